// Device code of the AR-Topk compressor for gfx950 (wave64).
//
// Kernels (in the order one step runs them):
//   k_fill_zero      clears the per-call scratch (histograms, scan flags, ...)
//   k_guess          (long flat vectors) samples g + residual and guesses a lower
//                    bound on the key of the k-th largest magnitude
//   k_pass_a         acc = g + residual in place, per-worker variance
//                    partials, and per-chunk 12-bit top-digit histograms of |acc|
//   k_pass_mark      the same pass behind k_guess: instead of histograms a bit
//                    mask of the keys reaching the guessed bound; its blocks
//                    stride over the tiles of the vector
//   k_guess_tiles / k_guess_segs, k_mark_tiles, k_tiles_pick .. k_tiles_out   the leader's own
//                    pass where it is known up front, and segments of long vectors: bounds,
//                    marked elements handed on tile by tile, and the selection from these
//   k_mark_spans     the marking alone, on vectors that are only read: their marked
//                    elements per span of a wave (k_spans_or_hist then writes the list)
//   k_hist0          the same histograms alone (stand-alone select, segments,
//                    after a guess that did not hold)
//   k_pass_seg       g + residual and those histograms in one pass, for the leader of a
//                    segmented step that is known up front
//   k_stats          variance partials alone (stand-alone variance)
//   k_squares        sums of squares of vectors and of their kept values
//   k_leader         finishes the variances and takes the first argmax
//   k_pick0          (flat VAR: finishes the variances, takes the leader;) finds the
//                    threshold digit and every chunk's list offset
//   k_pick_mask      the same first step when the fused pass left a mask: accepts
//                    the guessed bound or asks for the histogram route
//   k_compact1       ordered compaction of the leader's survivors, one block
//                    per chunk, no inter-block dependency
//   k_mask_or_hist   the survivor list written from the mask instead; or, after
//                    a guess that did not hold, k_hist0's work in the same launch
//   k_compact        ordered compaction with a decoupled look-back scan: the
//                    rarely needed deeper array pass
//   k_list_hist      digit histograms over the survivor list
//   k_level1 / k_level2 / k_final   the launches behind the first pick where
//                    alternatives exist: each does whichever of two jobs the state
//                    asks for (list histogram or array pass; final pass over the
//                    list or level-3 array pass writing the outputs), so that the
//                    rarely needed array passes cost no launches of their own
//   k_tile_starts    number of kept indices below every tile of a streaming pass
//   k_pass_rest      (leader known up front) EF add + gather + residual zeroing
//                    of all other workers in one streaming pass over the tiles
//   k_sum_update     (leader known up front) ordered sum over the workers' gathered
//                    rows and the dense update in one pass over the tiles
//   k_sum_rows       ordered sum over the workers' gathered rows
//   k_gather         vals / ordered sum / residual zeroing at the k indices
//   k_zero_at        residual zeroing alone
//   k_update_fill    dense update = zeros + k scattered sums, written once
//   k_small_step     a whole step on a short vector
//   k_update_tiles   the same for long, sparsely kept vectors: zeros streamed tile
//                    by tile, the sums stored behind them
//
// Keys are the 31 magnitude bits of the float32 (sign cleared), so integer
// order on keys is the order of |x|.  The radix digits are 12 + 12 + 7 bits.
//
// Chunks.  A vector range is cut into at most kMaxChunks contiguous chunks, each
// a whole number of 8192-element tiles.  The histogram pass stores, per chunk,
// the SUFFIX sums of its top-digit histogram: S[c][b] = number of keys of chunk
// c whose top digit is >= b.  Once the threshold digit b0 is known, S[c][b0] is
// exactly the number of survivors chunk c will emit, so an exclusive scan over
// the chunks gives every chunk its place in the survivor list and the big
// compaction pass needs no communication between blocks.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>
#include <stdint.h>
#include <limits.h>

namespace artopk {

constexpr int kMaxW = 64;
constexpr int kHistBins = 4096;          // 12-bit digits (the last digit uses 128 of them)
constexpr int kHistReps = 16;            // partial copies of a whole-vector histogram (spreads the atomics)
// One slot of whole-vector scratch (32-bit words): the partial histogram copies, then the
// histogram of the threshold-guess sample, then its control words.
constexpr int kSlotGuessHist = kHistReps * kHistBins;
constexpr int kSlotCtrl = kSlotGuessHist + kHistBins;  // [0] blocks done, [1] guessed key bound, [2] blocks of k_guess_tiles through
constexpr int kSlotMcount = kSlotCtrl + 16;            // marked elements per chunk, kMcountLine words apart
constexpr int kMcountLine = 16;  // (neighbouring chunks are marked at the same time, and additions to one line of memory wait
                                 // for each other: 138 M elements read only, one in 800 marked, 104 us side by side, 90 so)
constexpr int kSlotWords = kSlotMcount + 1024 * kMcountLine;
constexpr int kGuessMidAt = 8 * kHistBins;             // (k_guess_tiles: three histograms in copies' places)
constexpr int kGuessOddAt = 9 * kHistBins;
constexpr int kGuessLowAt = 10 * kHistBins;
constexpr uint32_t kNoGuess = 0xffffffffu;             // no key reaches this bound
constexpr int kGuessRun = 16;                          // consecutive elements per sample run
constexpr uint32_t kKeyMask = 0x7fffffffu;
constexpr uint32_t kQuotaInf = 0x7fffffffu;

// digit l (0,1,2) of a key: shift and mask
__host__ __device__ constexpr int digit_shift(int level) { return level == 0 ? 19 : (level == 1 ? 7 : 0); }
__host__ __device__ constexpr uint32_t digit_mask(int level) { return level == 2 ? 0x7fu : 0xfffu; }

// The pieces of k_mark_spans: the marked elements of every `span` elements, in order.
struct TileBuf {
  uint2* buf;       // [vector][span][cap] (index, raw bits)
  uint32_t* cnt;    // [vector][span] marked elements, which may be more than cap
  int64_t buf_stride;  // entries per vector
  int64_t cnt_stride;  // spans per vector
  int32_t cap;         // entries per span
  int32_t span;
};

struct PtrTable {
  float* p[kMaxW];
};

// Device-resident selection state; one per select in flight.
struct SelState {
  uint32_t lo, hi;         // candidate keys: lo <= key <= hi
  uint32_t n_gt;           // keys > hi inside the element range
  uint32_t need;           // entries still to be taken from the candidates (>= 1)
  uint32_t cand;           // number of candidate keys
  uint32_t level;          // radix digits resolved so far (0..3)
  uint32_t compact_level;  // level at which the survivor list was written (0 = not yet)
  uint32_t list_count;     // entries in the survivor list
  uint32_t use_mask;       // the list is written from the survivor bit mask of the fused pass
  uint32_t need_full;      // the guessed bound did not work out: the top-digit histogram of every key is needed
  uint32_t list_lo;        // with use_mask: the list holds every key >= list_lo (<= lo)
  uint32_t many;           // a short vector's threshold shares its top digit with many others (small_few); for select_info
  uint32_t pad[4];
};

// Bits of the sticky device-side error word.
constexpr uint32_t kErrPick = 1u;      // a histogram did not cover the wanted count
constexpr uint32_t kErrWait = 2u;      // a bounded look-back wait expired
constexpr uint32_t kErrSequence = 4u;  // a kernel found the state it needs missing
constexpr uint32_t kErrIndex = 8u;     // an index outside [0, N) reached gather / scatter

// Layout of one segment's zero-initialised scratch block (32-bit words).
constexpr int kSegState = 0;                       // SelState (16 words)
constexpr int kSegCounters = 16;                   // tile counters of the look-back passes (16 words)
constexpr int kSegHist1 = 32;                      // next-digit histogram, digit 1
constexpr int kSegHist2 = kSegHist1 + kHistBins;   // next-digit histogram, digit 2
constexpr int kSegHtop = kSegHist2 + kHistBins;    // top-digit histogram (when built by k_hist0)
constexpr int kSegWords = kSegHtop + kHistBins;
// Look-back flag words per 16384 elements: one of the array passes at level 2 and at level 3, four of the
// final list pass (whose tiles are 4096 entries).
constexpr int kNumLookback = 6;

struct ChunkGeom {
  int64_t chunk0;       // first element of chunk 0 (a multiple of kTile, <= range start)
  int64_t chunk_elems;  // elements per chunk (a multiple of kTile)
  int32_t nchunks;
};

// One selection problem: the k largest magnitudes of x[e_lo, e_hi).
struct SegDesc {
  int64_t e_lo, e_hi;
  ChunkGeom geom;      // chunk layout of the range
  int64_t koff;        // first slot of this segment in idx_out (and in the leader's vals row)
  int64_t list_base;   // first entry of this segment's survivor list (a multiple of 4)
  int64_t flag_base;   // first look-back tile of this segment
  int32_t chunk_begin; // first chunk slot of this segment in S / chunk_off
  uint32_t k;          // entries wanted
  uint32_t cap;        // survivor-list capacity of this segment
  int32_t vec;         // which vector of the pointer table to select on; -1 = the leader's
  // its tiles among those of the layout (see TileArgs), the blocks that have them, and further copies of its bins
  int32_t tile_begin, ntiles, group_begin, bins_begin, bins_more;
  int32_t hreps;  // k_hist0 adds the blocks' histograms to this many copies in SelParams::hcopies (1: to the
                  // one in the segment's scratch block)
};

// Everything the selection kernels need; blockIdx.y
// picks the segment.  With table == nullptr there is one segment, `one`.
struct SelParams {
  PtrTable tab;
  const int32_t* leader_dev;
  int64_t n;               // length of the vector
  uint32_t* hcopies;       // copies of top-digit histograms that k_hist0 fills (h_all's memory, when no pass fills that)
  int64_t hcopy_stride;    // their words per vector
  const uint32_t* h_all;   // [workers][kSlotWords] whole-vector histograms from the fused pass, or nullptr
  const uint64_t* mask;    // [workers][mask_stride] survivor bit masks from the fused pass, or nullptr
  int64_t mask_stride;     // 64-bit words per worker
  TileBuf tiles;           // pieces of a marking of vectors that are only read (buf == nullptr: none)
  int32_t use_mcount;      // the slots' per-chunk counts of marked elements are valid
  int32_t from_list;       // k_pick0: the top-digit histogram covers the survivor list written from the mask
  int32_t after_mask;      // k_pick0 behind k_mask_or_hist: from_list if the mask was used, else the full pick
  int32_t only_if_need_full;  // this launch runs only for segments whose state says need_full
  uint32_t* zero_base;     // [segments][kSegWords]
  uint64_t* flags;         // [tiles][kNumLookback]
  uint32_t* S;             // [slot][kMaxChunks][4096] per-chunk suffix histograms
  uint32_t* chunk_off;     // [chunks]
  uint2* list;             // survivor lists
  int32_t* idx_out;
  float* vals_row;         // leader's row of gathered values, or nullptr
  float* zero_vec;         // the selected vector itself if its kept entries are to become +0.0 on the way, or nullptr
  uint32_t* err;
  // Several whole vectors at once: segment s is vector s of the table with `one` for a descriptor, its own
  // list, look-back flags, chunk offsets and output row.
  int32_t batch;
  uint32_t k_all;          // entries kept of all segments or vectors together
  int64_t list_stride;     // list entries per vector
  int64_t flag_stride;     // look-back tiles per vector
  const SegDesc* table;
  // per-chunk kernels of a segmented selection run one block per chunk of the whole layout:
  // entry b = (segment << 16) | chunk within the segment; nullptr: grid = (chunks, segments)
  const uint32_t* chunk_map;
  int32_t slot_by_leader;  // S slot = index of the selected vector (histograms of all workers exist) or 0
  int32_t pad;
  SegDesc one;
};

// The (segment, chunk) a block of a per-chunk kernel works on.
__device__ __forceinline__ void block_chunk(const SelParams& p, int& seg, int& c) {
  if (p.chunk_map != nullptr) {
    const uint32_t m = p.chunk_map[blockIdx.x];
    seg = (int)(m >> 16);
    c = (int)(m & 0xffffu);
  } else {
    seg = (int)blockIdx.y;
    c = (int)blockIdx.x;
  }
}

struct SegView {
  SegDesc d;
  const float* x;  // the vector this segment selects on
  SelState* st;
  uint32_t* counters;
  uint32_t* hist1;
  uint32_t* hist2;
  uint32_t* htop;       // top-digit histogram of the selected vector's range: htop_reps partial copies to add up
  int htop_reps;
  uint32_t* hseg;       // the segment's own top-digit histogram (single copy), what k_hist0 fills without h_all
  const uint32_t* ctrl;  // control words of the vector's slot (guessed bound), or nullptr
  const uint64_t* mask;  // survivor bit mask of the vector, or nullptr
  const uint2* tbuf;     // the vector's pieces, or nullptr
  const uint32_t* tcnt;  // marked elements per span
  int32_t tcap;          // entries per piece
  const uint32_t* mcount;  // marked elements per chunk of the vector, kMcountLine words apart, or nullptr
  uint64_t* flags;
  uint32_t* S;
  uint32_t* chunk_off;
  uint2* list;
  int32_t* idx_out;
  float* vals_row;
};

// ---------------------------------------------------------------------------
// small helpers
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t lane_id() { return threadIdx.x & 63u; }

__device__ __forceinline__ uint32_t popc_lt(uint64_t mask) {
  // number of set bits of `mask` in lanes below the calling lane
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Stores that go through the XCD's own cache to where every XCD sees them.
template <typename V>
__device__ __forceinline__ void store_through(V* p, V v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Loads of what other blocks of the launch have stored so, or added up.  (An acquire fence and ordinary loads instead
// invalidate the XCD's cache once for every wave: 16 us a wait with 256 blocks of 512 threads.)
template <typename V>
__device__ __forceinline__ V load_through(const V* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  return v;  // valid in lane 0
}

// What the lanes that CTRL names hold, in the rows (of 16 lanes) that ROWS names; 0 where there is no such lane.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t from_lanes(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ uint64_t from_lanes(uint64_t v) {
  return ((uint64_t)from_lanes<CTRL, ROWS>((uint32_t)(v >> 32)) << 32) | from_lanes<CTRL, ROWS>((uint32_t)v);
}

// Inclusive prefix sums over the 64 lanes of a wave, all of which call it: 1, 2, 4 and 8 lanes down inside each row, then
// each odd row takes the last lane of the row before it, and the upper half the last lane of the lower.  Lanes read each
// other's registers; by way of on-chip memory (shuffles) each of the six steps waits for
// it: a step on 65537 x 2 took 18.4 us so, now 17.3, 1 M x 4 27.9 and 27.3, a selection of 138 M 163.9 and 162.4.
template <typename V>
__device__ __forceinline__ V wave_incl_scan(V v) {
  v += from_lanes<0x111, 0xf>(v);
  v += from_lanes<0x112, 0xf>(v);
  v += from_lanes<0x114, 0xf>(v);
  v += from_lanes<0x118, 0xf>(v);
  v += from_lanes<0x142, 0xa>(v);
  v += from_lanes<0x143, 0xc>(v);
  return v;
}
// What the last lane holds.
__device__ __forceinline__ uint32_t wave_last(uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)v, 63); }

__device__ __forceinline__ uint64_t wave_allsum_u64(uint64_t v) {
  v = wave_incl_scan(v);
  return ((uint64_t)wave_last((uint32_t)(v >> 32)) << 32) | wave_last((uint32_t)v);  // the total, in every lane
}

constexpr int kTile = 8192;       // chunk granularity (a quarter of a tile of the fused pass)
constexpr int kMaxChunks = 1024;  // chunks per vector range
static_assert(kSlotWords == kSlotMcount + kMaxChunks * kMcountLine, "one count per chunk");
constexpr int kPassTile = 32768;      // elements per block iteration of the streaming passes (1024 threads x 8 float4)
constexpr int kMaxPassBlocks = 4096;  // blocks per worker of a streaming pass that strides over tiles

typedef float v4f __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// Variance in one pass that no single element can spoil.  Every thread keeps, in
// float64, the count and the sums of (x - c) and (x - c)^2 of the values it sees,
// with a shift c of its own: the mean of the first four of them.  At the end of a
// block the threads re-base their sums (exactly: S' = S + n d, SS' = SS + d (2 S + n d),
// d = c - r) to the shift r of the block's first thread and add them up.  For any
// data, a block that sees m values has (mean - r)^2 <= (m / 4) variance of its
// values (Cauchy-Schwarz: r is the mean of four of them), so the cancellation of
// the shifted one-pass formula is bounded by the block's length and does not grow
// with an outlier or an offset.  The block's sums become (count n, mean, M2 = sum
// of squared deviations from its mean); the blocks' triples of one worker are
// combined the same way, with the mean of the worker's first block as the shift:
//     N = sum n_b, A = sum n_b (mean_b - r), B = sum (M2_b + n_b (mean_b - r)^2),
//     mean = r + A / N, M2 = B - A^2 / N.
// The order of every sum is fixed by the launch shape, so the result is reproducible.
// Partials layout: partials[w][0][b] = n_b, [w][1][b] = mean_b, [w][2][b] = M2_b.
// ---------------------------------------------------------------------------
struct VarAcc {
  double c = 0.0, s = 0.0, ss = 0.0;
  uint32_t cnt = 0u;
  // the shift is taken from the first group (or element) a thread sees: call seed before the
  // first add of every batch (it acts once)
  __device__ __forceinline__ void seed4(const v4f t) {
    if (cnt == 0u) c = (((double)t.x + (double)t.y) + ((double)t.z + (double)t.w)) * 0.25;
  }
  __device__ __forceinline__ void seed1(float x) {
    if (cnt == 0u) c = (double)x;
  }
  __device__ __forceinline__ void add4(const v4f t) {
    const double d0 = (double)t.x - c, d1 = (double)t.y - c, d2 = (double)t.z - c, d3 = (double)t.w - c;
    s += (d0 + d1) + (d2 + d3);
    ss = fma(d0, d0, ss);
    ss = fma(d1, d1, ss);
    ss = fma(d2, d2, ss);
    ss = fma(d3, d3, ss);
    cnt += 4u;
  }
  __device__ __forceinline__ void add1(float x) {
    const double d = (double)x - c;
    s += d;
    ss = fma(d, d, ss);
    cnt += 1u;
  }
};

__device__ __forceinline__ double wave_allsum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;  // the total, in every lane (the same bits: every lane adds the same pairs)
}

// Adds up the threads' sums of a block of T threads (all of them call it) and thread 0 writes
// the block's (n, mean, M2) to partials[w][.][b] (nblk blocks per worker).  Thread 0 must be a
// thread that saw a value whenever any thread of the block did (it owns the block's first group).
// THROUGH: for a reader in the same launch.
template <int T, bool THROUGH = false>
__device__ __forceinline__ void block_moments(const VarAcc& acc, double* __restrict__ partials, int w, int nblk,
                                              int b) {
  constexpr int NW = T / 64;
  __shared__ double red[3 * NW + 1];
  const int tid = threadIdx.x;
  if (tid == 0) red[3 * NW] = acc.c;
  __syncthreads();
  const double r = red[3 * NW];
  const double n_t = (double)acc.cnt;
  const double d = acc.cnt != 0u ? acc.c - r : 0.0;
  const double s = wave_sum(acc.s + n_t * d), ss = wave_sum(acc.ss + d * (2.0 * acc.s + n_t * d)), n = wave_sum(n_t);
  if ((tid & 63) == 0) {
    red[tid >> 6] = s;
    red[NW + (tid >> 6)] = ss;
    red[2 * NW + (tid >> 6)] = n;
  }
  __syncthreads();
  if (tid == 0) {
    double S1 = 0.0, S2 = 0.0, N = 0.0;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      S1 += red[i];
      S2 += red[NW + i];
      N += red[2 * NW + i];
    }
    double mean = 0.0, m2 = 0.0;
    if (N > 0.0) {
      const double sm = S1 / N;
      mean = r + sm;
      m2 = S2 - S1 * sm;
      if (m2 < 0.0) m2 = 0.0;  // rounding only (NaN stays NaN)
    }
    double* __restrict__ out = partials + (size_t)w * 3 * nblk + b;
    if (THROUGH) {
      store_through(out, N);
      store_through(out + nblk, mean);
      store_through(out + 2 * (size_t)nblk, m2);
    } else {
      out[0] = N;
      out[nblk] = mean;
      out[2 * (size_t)nblk] = m2;
    }
  }
}

// Variance of worker w from its blocks' partials; the 64 lanes of one wave call it, every lane
// returns the variance (population: M2 / N).
// THROUGH: written in the same launch.
template <bool THROUGH = false>
__device__ __forceinline__ double wave_variance(const double* __restrict__ partials, int w, int nblk) {
  auto get = [](const double* q) { return THROUGH ? load_through(q) : *q; };
  const int lane = threadIdx.x & 63;
  const double* __restrict__ pn = partials + (size_t)w * 3 * nblk;
  const double* __restrict__ pm = pn + nblk;
  const double* __restrict__ pq = pm + nblk;
  const double r = get(pm);
  double n = 0.0, a = 0.0, bq = 0.0;
  for (int b = lane; b < nblk; b += 512) {  // eight blocks' triples in flight per lane (absent ones add nothing)
    double nb[8], mb[8], qb[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int at = b + 64 * j < nblk ? b + 64 * j : lane;
      nb[j] = get(pn + at);
      mb[j] = get(pm + at);
      qb[j] = get(pq + at);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (b + 64 * j < nblk) {
        const double d = mb[j] - r;
        n += nb[j];
        a += nb[j] * d;
        bq += qb[j] + nb[j] * d * d;
      }
    }
  }
  n = wave_allsum(n);
  a = wave_allsum(a);
  bq = wave_allsum(bq);
  double v = 0.0;
  if (n > 0.0) v = (bq - a * (a / n)) / n;
  if (!(v > 0.0)) v = (v != v) ? v : 0.0;
  return v;
}

template <bool NT>
__device__ __forceinline__ v4f load4(const float* p) {
  return NT ? __builtin_nontemporal_load(reinterpret_cast<const v4f*>(p)) : *reinterpret_cast<const v4f*>(p);
}
template <bool NT>
__device__ __forceinline__ void store4(float* p, v4f v) {
  if (NT)
    __builtin_nontemporal_store(v, reinterpret_cast<v4f*>(p));
  else
    *reinterpret_cast<v4f*>(p) = v;
}

// Gradient element types: float32, or 16 bits widened exactly to float32 before use
// (bfloat16: the bits become the upper half of the float32; float16: hardware conversion).
constexpr int kGF32 = 0, kGBF16 = 1, kGF16 = 2;
constexpr int kGNone = 3;  // no gradient: the vector is only read

template <int GT>
__device__ __forceinline__ float widen16(uint32_t h) {  // h: the 16 bits in the low half
  if (GT == kGBF16) return __uint_as_float(h << 16);
  return (float)__builtin_bit_cast(_Float16, (unsigned short)h);
}

// Four consecutive gradient elements starting at element index e (a multiple of 4).
template <bool NT, int GT>
__device__ __forceinline__ v4f load4g(const float* base, int64_t e) {
  if (GT == kGF32) return load4<NT>(base + e);
  typedef uint32_t v2u __attribute__((ext_vector_type(2)));
  const v2u* p = reinterpret_cast<const v2u*>(reinterpret_cast<const unsigned short*>(base) + e);
  const v2u r = NT ? __builtin_nontemporal_load(p) : *p;
  v4f v;
  v.x = widen16<GT>(r.x & 0xffffu);
  v.y = widen16<GT>(r.x >> 16);
  v.z = widen16<GT>(r.y & 0xffffu);
  v.w = widen16<GT>(r.y >> 16);
  return v;
}

template <int GT>
__device__ __forceinline__ float load1g(const float* base, int64_t e) {
  if (GT == kGF32) return base[e];
  return widen16<GT>(reinterpret_cast<const unsigned short*>(base)[e]);
}

// Block-wide inclusive scans of one word per thread: a scan inside each
// wave, then the wave totals through `wtot` (T/64 words of shared memory that no
// thread still reads on entry).  Two barriers; `wtot` is free again on return.
// The exclusive value is the result minus the thread's own word.
template <int T>
__device__ __forceinline__ uint32_t block_suffix_incl(uint32_t v, uint32_t* wtot, uint32_t* total = nullptr) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t incl = wave_incl_scan(v), all = wave_last(incl), s = all - incl + v;
  if (lane == 0) wtot[wave] = all;
  __syncthreads();
  uint32_t add = 0u, tot = 0u;
#pragma unroll
  for (int i = 0; i < T / 64; ++i) {
    const uint32_t x = wtot[i];
    tot += x;
    if (i > wave) add += x;
  }
  __syncthreads();
  if (total) *total = tot;
  return s + add;
}

template <int T>
__device__ __forceinline__ uint32_t block_prefix_incl(uint32_t v, uint32_t* wtot, uint32_t* total = nullptr) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t s = wave_incl_scan(v);
  if (lane == 63) wtot[wave] = s;
  __syncthreads();
  uint32_t add = 0u, tot = 0u;
#pragma unroll
  for (int i = 0; i < T / 64; ++i) {
    const uint32_t x = wtot[i];
    tot += x;
    if (i < wave) add += x;
  }
  __syncthreads();
  if (total) *total = tot;
  return s + add;
}

// Adds the 4096-bin LDS histogram `lh` of a T-thread block to total[0..4096)
// and writes its suffix sums to dst[0..4096), unless that is nullptr.  `red` is T words of LDS.  All
// threads of the block must call it after their last histogram update.
template <int T>
__device__ __forceinline__ void flush_suffix_hist(uint32_t* lh, uint32_t* red, uint32_t* __restrict__ dst,
                                                  uint32_t* __restrict__ total) {
  constexpr int BPT = kHistBins / T;  // consecutive bins per thread (a multiple of 4)
  static_assert(BPT >= 4 && BPT % 4 == 0, "block size must divide 1024");
  const int t = threadIdx.x;
  __syncthreads();
  uint32_t v[BPT];
#pragma unroll
  for (int j = 0; j < BPT / 4; ++j) {
    const uint4 q = reinterpret_cast<const uint4*>(lh)[(BPT / 4) * t + j];
    v[4 * j + 0] = q.x;
    v[4 * j + 1] = q.y;
    v[4 * j + 2] = q.z;
    v[4 * j + 3] = q.w;
  }
  // the plain counts also go to the histogram of the whole range (few bins are occupied)
#pragma unroll
  for (int j = 0; j < BPT; ++j)
    if (v[j]) atomicAdd(&total[BPT * t + j], v[j]);
  if (dst == nullptr) return;
#pragma unroll
  for (int j = BPT - 2; j >= 0; --j) v[j] += v[j + 1];
  const uint32_t carry = block_suffix_incl<T>(v[0], red) - v[0];
#pragma unroll
  for (int j = 0; j < BPT / 4; ++j) {
    uint4 q;
    q.x = v[4 * j + 0] + carry;
    q.y = v[4 * j + 1] + carry;
    q.z = v[4 * j + 2] + carry;
    q.w = v[4 * j + 3] + carry;
    reinterpret_cast<uint4*>(dst)[(BPT / 4) * t + j] = q;
  }
}

// leader >= 0 overrides the device-resident leader (used by the block that has just computed it)
__device__ __forceinline__ SegView seg_view(const SelParams& p, int seg, int leader = -1) {
  SegView v;
  v.d = p.table ? p.table[seg] : p.one;
  if (p.batch) {
    v.d.vec = seg;
    v.d.koff = (int64_t)seg * (int64_t)v.d.k;
    v.d.list_base = (int64_t)seg * p.list_stride;
    v.d.flag_base = (int64_t)seg * p.flag_stride;
  }
  uint32_t* zb = p.zero_base + (size_t)seg * kSegWords;
  v.st = reinterpret_cast<SelState*>(zb + kSegState);
  v.counters = zb + kSegCounters;
  v.hist1 = zb + kSegHist1;
  v.hist2 = zb + kSegHist2;
  v.flags = p.flags + (size_t)v.d.flag_base * kNumLookback;
  const int vec = v.d.vec >= 0 ? v.d.vec : (leader >= 0 ? leader : *p.leader_dev);
  v.x = p.tab.p[vec];
  const size_t slot = p.slot_by_leader ? (size_t)vec : 0;  // histogram slot: per vector, or the only one
  v.htop = p.h_all ? const_cast<uint32_t*>(p.h_all) + slot * kSlotWords
                   : (v.d.hreps > 1 ? p.hcopies + slot * (size_t)p.hcopy_stride : zb + kSegHtop);
  v.htop_reps = p.h_all ? kHistReps : v.d.hreps;
  v.hseg = zb + kSegHtop;
  v.ctrl = p.h_all ? p.h_all + slot * kSlotWords + kSlotCtrl : nullptr;
  v.mask = p.mask ? p.mask + slot * (size_t)p.mask_stride : nullptr;
  v.tbuf = p.tiles.buf ? p.tiles.buf + slot * (size_t)p.tiles.buf_stride : nullptr;
  v.tcnt = p.tiles.buf ? p.tiles.cnt + slot * (size_t)p.tiles.cnt_stride : nullptr;
  v.tcap = p.tiles.cap;
  v.mcount = (p.h_all && p.use_mcount) ? p.h_all + slot * kSlotWords + kSlotMcount : nullptr;
  v.S = p.S + (slot * kMaxChunks + (size_t)v.d.chunk_begin) * kHistBins;
  v.chunk_off = p.chunk_off + (p.batch ? (size_t)seg * kMaxChunks : (size_t)v.d.chunk_begin);
  v.list = p.list + v.d.list_base;
  v.idx_out = p.idx_out + v.d.koff;
  v.vals_row = p.vals_row ? p.vals_row + v.d.koff : nullptr;
  return v;
}

// ---------------------------------------------------------------------------
// k_fill_zero : clears three word ranges (any may be empty); if leader_dev is
// given it also records a leader that the host already knows.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
k_fill_zero(uint32_t* __restrict__ p1, size_t words1, uint32_t* __restrict__ p2, size_t words2,
            uint32_t* __restrict__ p3, size_t words3, int32_t leader, int32_t* __restrict__ leader_dev, int32_t* __restrict__ leader_out) {
  if (leader_dev != nullptr && blockIdx.x == 0 && threadIdx.x == 0) {
    *leader_dev = leader;
    if (leader_out) *leader_out = leader;
  }
  const size_t stride = (size_t)gridDim.x * 256;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < words1; i += stride) p1[i] = 0u;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < words2; i += stride) p2[i] = 0u;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < words3; i += stride) p3[i] = 0u;
}

// ---------------------------------------------------------------------------
// k_pass_a : acc = g + residual (in place over residual), variance partials,
//            and the histograms the selection needs from this pass.
//   grid = (nchunks, W), block = T; block (c, w) owns chunk c of worker w.
//   HIST: 0 nothing for the selection, 1 only for worker `hist_worker` (slot 0),
//         2 for every worker (worker w in slot w): per-chunk top-digit suffix
//         histograms S[slot][c] and the whole-vector histogram of the slot.
//   STATS: 0 none, 1 variance partials of acc, 2 of the raw gradient g: the
//   block's (count, mean, sum of squared deviations) in float64 (see VarAcc).
//   NT: non-temporal loads of g and stores of acc.
//   S == nullptr: nobody needs counts per chunk; the blocks stride over the tiles instead, a few of them each.  With
//   chunks of one tile the counts were 4 % more to write and the additions to the whole-vector histograms what bound the
//   pass of many workers: 11.7 M x 8 311 us a step, now 287, 3 M x 4 106 and 82, 5 M x 16 433 and 249.
// ---------------------------------------------------------------------------
constexpr int kPassAUnroll = 4;

template <int STATS, int HIST, bool NT, int GT, int T, int U>
__global__ void __launch_bounds__(T)
k_pass_a(PtrTable g, PtrTable res, int64_t n, ChunkGeom geom, int hist_worker, uint32_t* __restrict__ S,
         uint32_t* __restrict__ h_all, double* __restrict__ partials) {
  constexpr bool LH = HIST != 0;  // an LDS histogram is built
  __shared__ __attribute__((aligned(16))) uint32_t lh[LH ? kHistBins : 4];
  __shared__ uint32_t red_u[LH ? T : 1];

  // with a known leader its blocks (the only ones that work for the selection) are dispatched first
  const int w = (HIST == 1) ? (int)((blockIdx.y + (unsigned)hist_worker) % gridDim.y) : (int)blockIdx.y;
  const int c = blockIdx.x;
  const int nblk = gridDim.x;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const float* __restrict__ gp = g.p[w];
  float* __restrict__ rp = res.p[w];
  const bool do_hist = (HIST == 2) || (HIST == 1 && w == hist_worker);
  const size_t slot = (HIST == 2) ? (size_t)w : 0;

  if (LH) {
    if (do_hist)
      for (int b = tid; b < kHistBins; b += T) lh[b] = 0u;
    __syncthreads();
  }

  const bool by_tile = S == nullptr;
  const int64_t c_lo = by_tile ? (int64_t)c * T * U * 4 : geom.chunk0 + (int64_t)c * geom.chunk_elems;
  int64_t c_hi = by_tile ? n : c_lo + geom.chunk_elems;
  if (c_hi > n) c_hi = n;
  const int64_t q_hi = c_hi >> 2;  // whole float4 groups of this chunk
  const int64_t step = by_tile ? (int64_t)nblk * T * U : (int64_t)T * U;

  VarAcc va;

  // One tile: U rows of T float4 groups; the wave's rows start at group qw (a multiple of 64).
  // FULL: every group of the wave's rows lies inside the chunk, so nothing is predicated.
  auto tile = [&](const int64_t qw, auto full_tag) {
    constexpr bool FULL = decltype(full_tag)::value;
    v4f a[U], b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      // groups outside the chunk re-read its last group (unused): no branch between the loads,
      // so that all of them are in flight together
      const int64_t q = qw + lane + u * T;
      const int64_t ql = (FULL || q < q_hi) ? q : q_hi - 1;
      a[u] = load4g<NT, GT>(gp, 4 * ql);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {  // (one array after the other: see k_pass_mark)
      const int64_t q = qw + lane + u * T;
      const int64_t ql = (FULL || q < q_hi) ? q : q_hi - 1;
      b[u] = load4<NT>(rp + 4 * ql);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t q = qw + lane + u * T;
      const bool valid = FULL || q < q_hi;
      if (valid) {
        v4f v;
        v.x = a[u].x + b[u].x;
        v.y = a[u].y + b[u].y;
        v.z = a[u].z + b[u].z;
        v.w = a[u].w + b[u].w;
        store4<NT>(rp + 4 * q, v);
        if (STATS) {  // of the raw gradient, or of the error-fed value
          if (u == 0) va.seed4(STATS == 2 ? a[u] : v);
          va.add4(STATS == 2 ? a[u] : v);
        }
        if (LH) {
          if (do_hist) {
            atomicAdd(&lh[(__float_as_uint(v.x) & kKeyMask) >> 19], 1u);
            atomicAdd(&lh[(__float_as_uint(v.y) & kKeyMask) >> 19], 1u);
            atomicAdd(&lh[(__float_as_uint(v.z) & kKeyMask) >> 19], 1u);
            atomicAdd(&lh[(__float_as_uint(v.w) & kKeyMask) >> 19], 1u);
          }
        }
      }
    }
  };

  // the loop runs on the wave's first group, so all 64 lanes stay together
  const int64_t qw0 = (c_lo >> 2) + __builtin_amdgcn_readfirstlane(tid - lane);
  int64_t qw = qw0;
  for (; qw + (int64_t)(U - 1) * T + 64 <= q_hi; qw += step) tile(qw, std::true_type{});
  if (qw < q_hi) tile(qw, std::false_type{});
  // scalar tail (n not a multiple of 4): the block that owns the last chunk, or the first one
  if (by_tile ? c == 0 : c_hi == n) {
    const int64_t j = (n >> 2) * 4 + tid;
    if (j < n) {
      const float gj = load1g<GT>(gp, j);
      const float v = gj + rp[j];
      rp[j] = v;
      if (STATS) {
        va.seed1(STATS == 2 ? gj : v);
        va.add1(STATS == 2 ? gj : v);
      }
      if (LH) {
        if (do_hist) atomicAdd(&lh[(__float_as_uint(v) & kKeyMask) >> 19], 1u);
      }
    }
  }

  if (STATS) block_moments<T>(va, partials, w, nblk, c);
  if (LH) {
    if (do_hist) {
      // many blocks add to the same few hundred bins: spread them over kHistReps partial copies
      flush_suffix_hist<T>(lh, red_u, by_tile ? nullptr : S + (slot * kMaxChunks + (size_t)c) * kHistBins,
                           h_all + slot * kSlotWords + (size_t)(c % kHistReps) * kHistBins);
    }
  }
}

// ---------------------------------------------------------------------------
// k_pass_mark : the fused pass of the route with a guessed threshold bound:
//   acc = g + residual (in place over residual), variance partials (STATS as in
//   k_pass_a), and, instead of histograms, one bit per element: elements whose
//   key reaches the guessed bound of the worker's slot are marked in the slot's
//   bit mask and counted per chunk of the selection's chunk layout.
//   grid = (gx, W'), block = T; block (b, y) works on worker y (slot y) and takes
//   the tiles b, b + gx, b + 2 gx, ... of T U float4 groups, so that at any time
//   the blocks in flight read and write one contiguous window of each array
//   (measured 4 to 10 % faster than one contiguous chunk per block).
//   Mask layout: for every row of 64 float4 groups four 64-bit words, word e,
//   bit l <=> element 4 (64 row + l) + e is marked; the words of a tile are
//   ordered so that each wave writes the 32 words of its 8 rows as one 256-byte
//   piece (mask_word() gives the place; 32-byte pieces per row cost the pass 4 %).
//   The n mod 4 elements behind the last whole group are counted (in the last
//   chunk) but have no mask bit.
//   Counts: every wave adds its tile's count to mcount[chunk of the tile] in the
//   slot (cleared beforehand); chunk_elems must be a whole number of tiles.
//   Variance partials: block b of worker y (see VarAcc).
//   PLAIN: no bound is read and nothing is counted: the error-feedback add and the
//   statistics in the same striding order, for a step whose selection builds its own
//   histograms afterwards (long segmented vectors).  The ballots and the mask words
//   (zero, but for Inf and NaN) stay: without them the same pass streamed slower on
//   8 x 1e9 elements, 16.6 against 16.1 ms.
// ---------------------------------------------------------------------------
// First of the four mask words of row `row` (256 elements) of a vector: tiles of 128 rows, inside a
// tile row r belongs to wave r mod 16 as its (r / 16)-th row.
__device__ __forceinline__ int64_t mask_word(int64_t row) {
  return (row >> 7) * 512 + (row & 15) * 32 + ((row >> 4) & 7) * 4;
}

template <int STATS, bool NT, int GT, int T, int U, bool PLAIN = false>
__global__ void __launch_bounds__(T)
k_pass_mark(PtrTable g, PtrTable res, int64_t n, int64_t chunk_elems, uint32_t* __restrict__ h_all,
            uint64_t* __restrict__ mask, int64_t mask_stride, double* __restrict__ partials) {
  const int w = blockIdx.y;
  const int bx = blockIdx.x;
  const int nblk = gridDim.x;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const float* __restrict__ gp = g.p[w];
  float* __restrict__ rp = res.p[w];
  uint32_t* __restrict__ slot = h_all + (size_t)w * kSlotWords;
  uint32_t* __restrict__ mcount = slot + kSlotMcount;
  uint64_t* __restrict__ mrow = mask + (size_t)w * (size_t)mask_stride;

  // Marked <=> not (|acc| < bound): the same as key >= bound on the magnitude bits, NaNs included.
  const uint32_t gkey = PLAIN ? kNoGuess : slot[kSlotCtrl + 1];
  const float gf = gkey != kNoGuess ? __uint_as_float(gkey) : __builtin_inff();

  const int64_t q_hi = n >> 2;  // whole float4 groups of the vector
  constexpr int64_t TQ = (int64_t)T * U;  // groups per tile
  const int64_t ntiles = (q_hi + TQ - 1) / TQ;

  VarAcc va;
  const int wave_first = __builtin_amdgcn_readfirstlane(tid - lane);
  static_assert(T == 1024 && U == 8, "mask_word() is laid out for 16 waves x 8 rows");
  // One tile: U rows of T float4 groups; the wave's rows start at group qw (a multiple of 64).
  // FULL: every group of the tile lies inside the vector, so nothing is predicated.
  auto tile = [&](const int64_t qw, auto full_tag) {
    constexpr bool FULL = decltype(full_tag)::value;
    v4f a[U], b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      // groups outside the vector re-read its last group (unused): no branch between the loads,
      // so that all of them are in flight together
      const int64_t q = qw + lane + u * T;
      const int64_t ql = (FULL || q < q_hi) ? q : q_hi - 1;
      a[u] = load4g<NT, GT>(gp, 4 * ql);
    }
    // The tile's gradient loads first, then its residual loads: issued alternately (g, r, g, r, ...)
    // the same pass took 16.04 instead of 15.72 ms on 8 x 1e9 elements (residual first: 15.77).
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t q = qw + lane + u * T;
      const int64_t ql = (FULL || q < q_hi) ? q : q_hi - 1;
      b[u] = load4<NT>(rp + 4 * ql);
    }
    uint32_t marked = 0u;  // of this wave in this tile
    uint64_t mine = 0ull;  // lane 4 u + e keeps word e of the wave's row u
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t q = qw + lane + u * T;
      const bool valid = FULL || q < q_hi;
      v4f v = {0.f, 0.f, 0.f, 0.f};
      if (valid) {
        v.x = a[u].x + b[u].x;
        v.y = a[u].y + b[u].y;
        v.z = a[u].z + b[u].z;
        v.w = a[u].w + b[u].w;
        store4<NT>(rp + 4 * q, v);
        if (STATS) {  // of the raw gradient, or of the error-fed value
          if (u == 0) va.seed4(STATS == 2 ? a[u] : v);
          va.add4(STATS == 2 ? a[u] : v);
        }
      }
      const uint64_t m0 = __ballot(valid && !(__builtin_fabsf(v.x) < gf));
      const uint64_t m1 = __ballot(valid && !(__builtin_fabsf(v.y) < gf));
      const uint64_t m2 = __ballot(valid && !(__builtin_fabsf(v.z) < gf));
      const uint64_t m3 = __ballot(valid && !(__builtin_fabsf(v.w) < gf));
      marked += (uint32_t)(__popcll(m0) + __popcll(m1) + __popcll(m2) + __popcll(m3));
      mine = lane == 4 * u + 0 ? m0 : mine;
      mine = lane == 4 * u + 1 ? m1 : mine;
      mine = lane == 4 * u + 2 ? m2 : mine;
      mine = lane == 4 * u + 3 ? m3 : mine;
    }
    // rows behind the vector's end get zero words: the mask holds whole tiles
    if (lane < 4 * U) mrow[mask_word(qw >> 6) + lane] = mine;
    return marked;
  };

  for (int64_t ti = bx; ti < ntiles; ti += nblk) {
    const int64_t qw = ti * TQ + wave_first;  // wave-uniform, so all 64 lanes stay together (the masks need that)
    const uint32_t marked = (ti + 1) * TQ <= q_hi ? tile(qw, std::true_type{}) : tile(qw, std::false_type{});
    if (!PLAIN && lane == 0 && marked != 0u) atomicAdd(&mcount[(ti * TQ * 4) / chunk_elems * kMcountLine], marked);
  }
  // scalar tail (n not a multiple of 4): the first block
  if (bx == 0) {
    const int64_t j = q_hi * 4 + tid;
    if (j < n) {
      const float gj = load1g<GT>(gp, j);
      const float v = gj + rp[j];
      rp[j] = v;
      if (STATS) {
        va.seed1(STATS == 2 ? gj : v);
        va.add1(STATS == 2 ? gj : v);
      }
      if (!PLAIN && !(__builtin_fabsf(v) < gf)) atomicAdd(&mcount[(n - 1) / chunk_elems * kMcountLine], 1u);
    }
  }

  if (STATS) block_moments<T>(va, partials, w, nblk, bx);
}

// ---------------------------------------------------------------------------
// k_stats : the variances' part of read-only vectors in float64, grid = (nblk, W): the block's (count, mean, sum of
// squared deviations), see VarAcc.  Rows must be 16-byte aligned.
//   NT: non-temporal loads, for vectors that together are larger than twice the last-level
// cache: what earlier kernels left there (written and half-written lines) slowed ordinary
// loads to 4.4 TB/s on 2 x 138 M elements behind a residual rewrite, non-temporal ones
// run at 5.6 (253 against 200 us; 4 x 138 M alone 383 against 343).  Where the vectors
// partly lie in the cache ordinary loads are the better ones (1 x 60 M behind a rewrite:
// 54 against 92 us, 8 x 11.7 M 86 against 99, 1 x 138 M the same).
// ---------------------------------------------------------------------------
template <bool NT>
__global__ void __launch_bounds__(256)
k_stats(PtrTable x, int64_t n, double* __restrict__ partials) {
  const int w = blockIdx.y, bx = blockIdx.x, nblk = gridDim.x, tid = threadIdx.x;
  const float* __restrict__ xp = x.p[w];
  const int64_t n4 = n >> 2;
  VarAcc va;
  const int64_t tile = 256 * kPassAUnroll;
  const int64_t ntile = (n4 + tile - 1) / tile;
  for (int64_t t = bx; t < ntile; t += nblk) {
    const int64_t q0 = t * tile + tid;
    v4f a[kPassAUnroll];
#pragma unroll
    for (int u = 0; u < kPassAUnroll; ++u) {
      const int64_t q = q0 + u * 256;
      if (q < n4) a[u] = load4<NT>(xp + 4 * q);
    }
#pragma unroll
    for (int u = 0; u < kPassAUnroll; ++u) {
      const int64_t q = q0 + u * 256;
      if (q < n4) {
        if (u == 0) va.seed4(a[u]);
        va.add4(a[u]);
      }
    }
  }
  // elements not covered by whole float4 groups
  for (int64_t j = n4 * 4 + (int64_t)bx * 256 + tid; j < n; j += (int64_t)nblk * 256) {
    va.seed1(xp[j]);
    va.add1(xp[j]);
  }
  block_moments<256>(va, partials, w, nblk, bx);
}

// ---------------------------------------------------------------------------
// k_squares : sums of squares in float64 of w short rows of k values (of any alignment), which nfew blocks a row take, and
// in the blocks behind them of w vectors of n elements (16-byte aligned), which nblk take; part_few[w][nfew] and
// part_vec[w][nblk].  NT as in k_stats.  In one launch the rows are summed beside the vectors, and eight values a thread
// are on their way at a time: 2 x 138 M and 2 x 1.4 M 198 + 9 us in two, now 199; eight rows of 256 thousand 6.9 us one
// value after the other, now 4.8.  The long vectors are bound by memory (5.6 TB/s behind the residual rewrite).
// ---------------------------------------------------------------------------
template <bool NT>
__global__ void __launch_bounds__(256)
k_squares(PtrTable x, int64_t n, int nblk, PtrTable few, int64_t k, int nfew, double* __restrict__ part_vec,
          double* __restrict__ part_few) {
  __shared__ double red[4];
  const int w = blockIdx.y, tid = threadIdx.x;
  const bool rows = (int)blockIdx.x < nfew;
  const int bx = rows ? (int)blockIdx.x : (int)blockIdx.x - nfew, blocks = rows ? nfew : nblk;
  const float* __restrict__ xp = rows ? few.p[w] : x.p[w];
  const int64_t len = rows ? k : n;
  const int64_t n4 = rows ? 0 : n >> 2;
  double ss = 0.0;
  auto add = [&](float v) {
    const double d = (double)v;
    ss = fma(d, d, ss);
  };
  const int64_t tile = 256 * kPassAUnroll;
  const int64_t ntile = (n4 + tile - 1) / tile;
  for (int64_t t = bx; t < ntile; t += blocks) {
    const int64_t q0 = t * tile + tid;
    v4f a[kPassAUnroll];
#pragma unroll
    for (int u = 0; u < kPassAUnroll; ++u) {
      const int64_t q = q0 + u * 256;
      if (q < n4) a[u] = load4<NT>(xp + 4 * q);
    }
#pragma unroll
    for (int u = 0; u < kPassAUnroll; ++u) {
      if (q0 + u * 256 < n4) {
        add(a[u].x);
        add(a[u].y);
        add(a[u].z);
        add(a[u].w);
      }
    }
  }
  const int64_t step = (int64_t)blocks * 256;
  for (int64_t j = n4 * 4 + (int64_t)bx * 256 + tid; j < len; j += 8 * step) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = xp[j + u * step < len ? j + u * step : j];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (j + u * step < len) add(v[u]);
  }
  ss = wave_sum(ss);
  if ((tid & 63) == 0) red[tid >> 6] = ss;
  __syncthreads();
  if (tid == 0) (rows ? part_few : part_vec)[(size_t)w * blocks + bx] = (red[0] + red[1]) + (red[2] + red[3]);
}

// Sum of `count` partial sums; the 64 lanes of a wave call it, lane 0 has the result.
__device__ __forceinline__ double wave_total(const double* __restrict__ part, int count) {
  double v = 0.0;
  for (int b = threadIdx.x & 63; b < count; b += 512) {  // eight in flight
    double q[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) q[u] = part[b + 64 * u < count ? b + 64 * u : b];
#pragma unroll
    for (int u = 0; u < 8; ++u) v += b + 64 * u < count ? q[u] : 0.0;
  }
  return wave_sum(v);
}

// ---------------------------------------------------------------------------
// k_gain : one block.  gain_w = V_w / (V_w + R_w) with V_w, R_w the sums of squares of worker w's
// gathered values and of its residual after the step; the two have disjoint support, so V_w + R_w is
// the squared norm of the error-fed gradient.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(1024)
k_gain(const double* __restrict__ part_vals, int nblk_vals, const double* __restrict__ part_res, int nblk_res,
       int w_count, double* __restrict__ gain_out) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int w = wave; w < w_count; w += 16) {
    const double v = wave_total(part_vals + (size_t)w * nblk_vals, nblk_vals);
    const double r = wave_total(part_res + (size_t)w * nblk_res, nblk_res);
    if (lane == 0) gain_out[w] = (v + r > 0.0) ? v / (v + r) : 0.0;
  }
}

// ---------------------------------------------------------------------------
// k_sqnorm : one block.  out[w] = sum of the partial sums of squares of vector w;
// argmax = first w with the largest value (also stored as leader).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(1024)
k_sqnorm(const double* __restrict__ part, int nblk, int w_count, double* __restrict__ scratch,
         double* __restrict__ out, int32_t* __restrict__ leader_dev, int32_t* __restrict__ argmax_out) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int w = wave; w < w_count; w += 16) {
    const double v = wave_total(part + (size_t)w * nblk, nblk);
    if (lane == 0) {
      scratch[w] = v;
      if (out) out[w] = v;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int best = 0;
    for (int w = 1; w < w_count; ++w)
      if (scratch[w] > scratch[best]) best = w;
    if (leader_dev) *leader_dev = best;
    if (argmax_out) *argmax_out = best;
  }
}

__global__ void __launch_bounds__(256)
k_copy_i32(const int32_t* __restrict__ src_rows, const int32_t* __restrict__ row_dev, int64_t k,
           int32_t* __restrict__ dst) {
  const int64_t m = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (m < k) dst[m] = src_rows[(size_t)(*row_dev) * (size_t)k + (size_t)m];
}

// ---------------------------------------------------------------------------
// k_apply_update : w[idx[m]] = w[idx[m]] - eta * sum[m] (one float32 multiply,
// one float32 subtract), the sparse form of the model update.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
k_apply_update(float* __restrict__ weights, int64_t n, const int32_t* __restrict__ idx,
               const float* __restrict__ sum, int64_t k, float eta, uint32_t* __restrict__ err) {
  const int64_t m = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (m >= k) return;
  const int64_t i = (int64_t)idx[m];
  if (i < 0 || i >= n) {
    atomicOr(err, kErrIndex);
    return;
  }
  const float step = eta * sum[m];
  weights[i] = weights[i] - step;
}

// ---------------------------------------------------------------------------
// k_leader : one block of 1024 threads.  Merges the per-block moments of every
// worker in a fixed order, var_w = M2 / n, leader = first argmax.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(1024)
k_leader(const double* __restrict__ partials, int w_count, int nblk, int64_t n,
         double* __restrict__ var_scratch, double* __restrict__ var_out,
         int32_t* __restrict__ leader_dev, int32_t* __restrict__ leader_out) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  for (int w = wave; w < w_count; w += 16) {
    const double v = wave_variance(partials, w, nblk);
    if (lane == 0) {
      var_scratch[w] = v;
      if (var_out) var_out[w] = v;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int best = 0;
    for (int w = 1; w < w_count; ++w)
      if (var_scratch[w] > var_scratch[best]) best = w;
    *leader_dev = best;
    if (leader_out) *leader_out = best;
  }
}

__global__ void k_set_leader(int32_t leader, int32_t* __restrict__ leader_dev, int32_t* __restrict__ leader_out) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    *leader_dev = leader;
    if (leader_out) *leader_out = leader;
  }
}

// The round-robin leader from the iteration counter kept on the device (Alg. 1,
// STAR branch): leader = counter mod w, then the counter moves on by one.
__global__ void k_counter_leader(uint64_t* __restrict__ counter, int32_t w, int32_t* __restrict__ leader_dev,
                                 int32_t* __restrict__ leader_out) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    const uint64_t c = *counter;
    const int32_t leader = (int32_t)(c % (uint64_t)w);
    *leader_dev = leader;
    if (leader_out) *leader_out = leader;
    *counter = c + 1u;
  }
}

__global__ void k_set_counter(uint64_t* __restrict__ counter, uint64_t value) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *counter = value;
}

// words of a segment's scratch block, behind the last digit's 128 counts in kSegHist2: what the marking of tiles goes by
constexpr int kTileInfo = kSegHist2 + 1024;
constexpr int kTileBound = 0;  // the bound (0: none)
constexpr int kTileShift = 1;  // bits of a bin
constexpr int kTileZero = 2;   // marked keys from here on are stored as +0.0 at once
constexpr int kTileFull = 8;   // (of the first segment's) some segment's bound does not hold
constexpr int kMarkThreads = 512, kMarkTile = 32 * kMarkThreads;  // a block of k_mark_tiles, and what it loads at a time
constexpr int kMarkMax = 2816;   // entries a tile's piece can have (22 KiB on chip: four blocks a compute unit)
constexpr int kTileBins = 4095;  // bins that start at the bound; what is above them all is not binned

// bound: at most k keys of the sample's share, and a margin, reach it; mid: the sample's estimate of the threshold; top: a
// digit that surely lies above it.
__device__ __forceinline__ void tile_info(uint32_t* __restrict__ info, uint32_t bound, uint32_t mid, uint32_t top) {
  if (bound == 0u) return;
  const uint32_t reach = ((top + 1u) << 19) - bound;
  uint32_t s = 0u;
  while (s < 19u && ((uint32_t)kTileBins << s) < reach) ++s;
  info[kTileBound] = bound;
  info[kTileShift] = s;
  info[kTileZero] = mid < bound ? bound : mid < 0x7f800000u ? mid : 0x7f800000u;
}

// ---------------------------------------------------------------------------
// k_guess : a lower bound on the key of the k-th largest |g + residual| of each
// vector, from a sample, before the fused pass runs.  grid = (blocks, vectors),
// block = 256; vector y uses slot y.  The sample is `runs` runs of kGuessRun
// consecutive elements, run r starting at (r stride) rounded down to a multiple
// of kGuessRun.  The last block to finish takes the top digit d of the sample's
// m_hi-th largest key and publishes d << 19 (kNoGuess if the sample is smaller
// than m_hi, or more than m_max of its keys reach that bound).  GT = kGNone samples
// the residuals alone.  The bound is only a guess: whoever uses it checks that at least
// k keys of the whole vector reach it.
// ---------------------------------------------------------------------------
template <int GT>
__global__ void __launch_bounds__(256)
k_guess(PtrTable g, PtrTable res, uint32_t* __restrict__ slots, int runs, int64_t stride, uint32_t m_hi,
        uint32_t m_max) {
  __shared__ uint32_t lh[kHistBins];
  __shared__ uint32_t wsum[4];
  __shared__ int last_sh, hit_sh;
  const int tid = threadIdx.x;
  const int v = blockIdx.y;
  const float* __restrict__ gp = g.p[v];
  const float* __restrict__ rp = res.p[v];
  uint32_t* __restrict__ ghist = slots + (size_t)v * kSlotWords + kSlotGuessHist;
  uint32_t* __restrict__ ctrl = slots + (size_t)v * kSlotWords + kSlotCtrl;
  for (int b = tid; b < kHistBins; b += 256) lh[b] = 0u;
  __syncthreads();
  for (int r = blockIdx.x * 256 + tid; r < runs; r += gridDim.x * 256) {
    const int64_t e0 = ((int64_t)r * stride) & ~(int64_t)(kGuessRun - 1);
    v4f a[kGuessRun / 4], b[kGuessRun / 4];
#pragma unroll
    for (int i = 0; i < kGuessRun / 4; ++i) {
      if (GT != kGNone) a[i] = load4g<false, GT>(gp, e0 + 4 * i);
      b[i] = load4<false>(rp + e0 + 4 * i);
    }
#pragma unroll
    for (int i = 0; i < kGuessRun / 4; ++i) {
      atomicAdd(&lh[(__float_as_uint(GT != kGNone ? a[i].x + b[i].x : b[i].x) & kKeyMask) >> 19], 1u);
      atomicAdd(&lh[(__float_as_uint(GT != kGNone ? a[i].y + b[i].y : b[i].y) & kKeyMask) >> 19], 1u);
      atomicAdd(&lh[(__float_as_uint(GT != kGNone ? a[i].z + b[i].z : b[i].z) & kKeyMask) >> 19], 1u);
      atomicAdd(&lh[(__float_as_uint(GT != kGNone ? a[i].w + b[i].w : b[i].w) & kKeyMask) >> 19], 1u);
    }
  }
  __syncthreads();
  for (int b = tid; b < kHistBins; b += 256) {
    const uint32_t c = lh[b];
    if (c) atomicAdd(&ghist[b], c);
  }
  // (what this wave has added is there: see meet_arrive; a fence would write back and invalidate the cache for every wave)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) {
    last_sh = __hip_atomic_fetch_add(&ctrl[0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1 ? 1 : 0;
    hit_sh = -1;
  }
  __syncthreads();
  if (!last_sh) return;
  // the last block: suffix sums over the sample histogram, 16 consecutive bins per thread
  uint32_t h[16];
  uint32_t tot = 0u;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    h[j] = __hip_atomic_load(&ghist[16 * tid + j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    tot += h[j];
  }
  // inclusive suffix sum of tot over the 64 lanes, then over the 4 waves
  const uint32_t incl = wave_incl_scan(tot);
  const uint32_t suf = wave_last(incl) - incl + tot;
  if ((tid & 63) == 0) wsum[tid >> 6] = suf;
  __syncthreads();
  uint32_t above = suf - tot;  // bins of higher threads in this wave
  for (int i = (tid >> 6) + 1; i < 4; ++i) above += wsum[i];
#pragma unroll
  for (int j = 15; j >= 0; --j) {
    if (above < m_hi && above + h[j] >= m_hi) {  // one thread, one bin
      // (a bound that so many keys reach that the list could not take them is none)
      if (above + h[j] <= m_max) hit_sh = 16 * tid + j;
    }
    above += h[j];
  }
  __syncthreads();
  const int hit = hit_sh;
  // bounds above infinity's digit would not survive the floating-point comparison of the fused pass
  const uint32_t bound = hit >= 0 ? (uint32_t)(hit < 0xff0 ? hit : 0xff0) << 19 : kNoGuess;
  if (tid == 0) ctrl[1] = bound;
}

// ---------------------------------------------------------------------------
// k_hist0 : per-chunk top-digit suffix histograms of |x[e_lo .. e_hi)| for the
// leader's vector.  grid = (max chunks of a segment, segments), block = T (1024:
// there are at most about a thousand blocks, so a block must keep many loads in flight:
// eight float4 groups a thread, unconditional; four behind conditions took 137 us on
// 138 M elements, these 116).  Whole float4 groups of the chunk are read as such, the at
// most three elements before and behind them one by one.  Bound by the chip's memory and
// then by the on-chip atomics (more copies of the block's histogram changed nothing).
// ---------------------------------------------------------------------------
template <int T>
__device__ __forceinline__ void hist0_body(const SelParams& p) {
  constexpr int U = 8;  // float4 groups a thread has in flight
  __shared__ __attribute__((aligned(16))) uint32_t lh[kHistBins];
  __shared__ uint32_t red_u[T];
  int seg, c;
  block_chunk(p, seg, c);
  const SegView sv = seg_view(p, seg);
  if (c >= sv.d.geom.nchunks) return;
  if (p.only_if_need_full && sv.st->need_full == 0u) return;
  const int tid = threadIdx.x;
  const float* __restrict__ xp = sv.x;
  for (int b = tid; b < kHistBins; b += T) lh[b] = 0u;
  __syncthreads();
  int64_t cs = sv.d.geom.chunk0 + (int64_t)c * sv.d.geom.chunk_elems;
  int64_t ce = cs + sv.d.geom.chunk_elems;
  if (cs < sv.d.e_lo) cs = sv.d.e_lo;
  if (ce > sv.d.e_hi) ce = sv.d.e_hi;
  auto count = [&](uint32_t raw) { atomicAdd(&lh[(raw & kKeyMask) >> 19], 1u); };
  const int64_t q_lo = (cs + 3) >> 2, q_hi = ce >> 2;  // whole float4 groups of the chunk
  if (q_lo < q_hi) {
    int64_t q0 = q_lo;
    for (; q0 + T * U <= q_hi; q0 += T * U) {
      uint4 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = *reinterpret_cast<const uint4*>(xp + 4 * (q0 + tid + u * T));
#pragma unroll
      for (int u = 0; u < U; ++u) {
        count(v[u].x);
        count(v[u].y);
        count(v[u].z);
        count(v[u].w);
      }
    }
    if (q0 < q_hi) {
      uint4 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {  // (no branch around the loads: behind the chunk they re-read its last group)
        const int64_t q = q0 + tid + u * T;
        v[u] = *reinterpret_cast<const uint4*>(xp + 4 * (q < q_hi ? q : q_hi - 1));
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (q0 + tid + u * T < q_hi) {
          count(v[u].x);
          count(v[u].y);
          count(v[u].z);
          count(v[u].w);
        }
      }
    }
    // the chunk's first and last elements outside whole groups (at most three each)
    const int64_t j = tid < 4 ? cs + tid : 4 * q_hi + (tid - 4);
    if (tid < 8 && j < (tid < 4 ? 4 * q_lo : ce)) count(__float_as_uint(xp[j]));
  } else if (cs + tid < ce) {  // not one whole group: at most six elements
    count(__float_as_uint(xp[cs + tid]));
  }
  flush_suffix_hist<T>(lh, red_u, sv.S + (size_t)c * kHistBins,
                       sv.htop + (size_t)(c % sv.htop_reps) * kHistBins);
}

// ---------------------------------------------------------------------------
// k_pass_seg : the leader's fused pass of a segmented step whose leader is known up front:
// acc = g + residual in place, chunk by chunk of the segments' layout, and k_hist0's
// per-chunk histograms of the result in the same read.  One block per chunk, as k_hist0.
// Striding over the tiles instead and reading the vector again for the histograms takes longer:
// the whole step on 200 k x 4 in 20 segments 67 us, now 55.  (Long vectors go by tiles.)
// ---------------------------------------------------------------------------
template <bool NT, int GT, int T>
__global__ void __launch_bounds__(T)
k_pass_seg(SelParams p, const float* __restrict__ g, float* __restrict__ r) {
  constexpr int U = 8;
  __shared__ __attribute__((aligned(16))) uint32_t lh[kHistBins];
  __shared__ uint32_t red_u[T];
  int seg, c;
  block_chunk(p, seg, c);
  const SegView sv = seg_view(p, seg);
  if (c >= sv.d.geom.nchunks) return;
  const int tid = threadIdx.x;
  for (int b = tid; b < kHistBins; b += T) lh[b] = 0u;
  __syncthreads();
  int64_t cs = sv.d.geom.chunk0 + (int64_t)c * sv.d.geom.chunk_elems;
  int64_t ce = cs + sv.d.geom.chunk_elems;
  if (cs < sv.d.e_lo) cs = sv.d.e_lo;
  if (ce > sv.d.e_hi) ce = sv.d.e_hi;
  auto count = [&](float v) { atomicAdd(&lh[(__float_as_uint(v) & kKeyMask) >> 19], 1u); };
  auto single = [&](int64_t j) {
    const float v = load1g<GT>(g, j) + r[j];
    r[j] = v;
    count(v);
  };
  const int64_t q_lo = (cs + 3) >> 2, q_hi = ce >> 2;  // whole float4 groups of the chunk
  if (q_lo < q_hi) {
    auto tile = [&](int64_t q0, auto full_tag) {
      constexpr bool FULL = decltype(full_tag)::value;
      v4f a[U], b[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {  // (groups behind the chunk re-read its last one, unused)
        const int64_t q = q0 + tid + u * T;
        a[u] = load4g<NT, GT>(g, 4 * (FULL || q < q_hi ? q : q_hi - 1));
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t q = q0 + tid + u * T;
        b[u] = load4<NT>(r + 4 * (FULL || q < q_hi ? q : q_hi - 1));
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t q = q0 + tid + u * T;
        if (FULL || q < q_hi) {
          v4f v;
          v.x = a[u].x + b[u].x;
          v.y = a[u].y + b[u].y;
          v.z = a[u].z + b[u].z;
          v.w = a[u].w + b[u].w;
          store4<NT>(r + 4 * q, v);
          count(v.x);
          count(v.y);
          count(v.z);
          count(v.w);
        }
      }
    };
    int64_t q0 = q_lo;
    for (; q0 + T * U <= q_hi; q0 += T * U) tile(q0, std::true_type{});
    if (q0 < q_hi) tile(q0, std::false_type{});
    // the chunk's first and last elements outside whole groups (at most three each)
    const int64_t j = tid < 4 ? cs + tid : 4 * q_hi + (tid - 4);
    if (tid < 8 && j < (tid < 4 ? 4 * q_lo : ce)) single(j);
  } else if (cs + tid < ce) {  // not one whole group: at most six elements
    single(cs + tid);
  }
  flush_suffix_hist<T>(lh, red_u, sv.S + (size_t)c * kHistBins,
                       sv.htop + (size_t)(c % sv.htop_reps) * kHistBins);
}

template <int T>
__global__ void __launch_bounds__(T)
k_hist0(SelParams p) {
  hist0_body<T>(p);
}

// ---------------------------------------------------------------------------
// Selection state machine.  k_pick0 writes the state after the top digit (level
// 1) and decides whether the level-1 survivors fit the list.  Nothing else
// writes the state: later kernels replay the remaining digit picks from the
// next-digit histograms in their prologue (derive_state), every block for
// itself -- the result is a pure function of hist1 / hist2, so all blocks agree
// and no extra launches are needed.
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool fits_list(const SelState& st, uint32_t cap) {
  return (uint64_t)st.n_gt + (uint64_t)st.cand <= (uint64_t)cap;
}

// Narrows st (in shared memory) by digit `digit` (1 or 2); thread t holds the counts of the bins BPT t .. of
// that digit over the current candidates.  All T threads call it; `part` is T words of shared memory.
template <int T>
__device__ void block_pick_bins(SelState& st, const uint32_t (&h)[kHistBins / T], int digit, uint32_t* part,
                                uint32_t* __restrict__ err) {
  constexpr int BPT = kHistBins / T;
  const int t = threadIdx.x;
  uint32_t tot = 0u;
#pragma unroll
  for (int j = 0; j < BPT; ++j) tot += h[j];
  __syncthreads();  // st is stable and `part` is free
  uint32_t total;
  uint32_t above = block_suffix_incl<T>(tot, part, &total) - tot;
  const uint32_t need = st.need;
  int hit = -1;
  uint32_t hit_above = 0u, hit_cnt = 0u;
#pragma unroll
  for (int j = BPT - 1; j >= 0; --j) {
    if (hit < 0 && above < need && need <= above + h[j]) {
      hit = BPT * t + j;
      hit_above = above;
      hit_cnt = h[j];
    }
    above += h[j];
  }
  __syncthreads();  // every thread has read st.need
  if (hit >= 0) {   // exactly one thread when the histogram holds >= need keys
    const int sh = digit_shift(digit);
    st.lo = st.lo | ((uint32_t)hit << sh);
    st.hi = st.lo | ((1u << sh) - 1u);
    st.n_gt += hit_above;
    st.need -= hit_above;
    st.cand = hit_cnt;
    st.level = (uint32_t)digit + 1u;
  }
  if (t == 0 && total < need) atomicOr(err, kErrPick);  // histogram does not cover `need`
  __syncthreads();
}

// The same with the digit's histogram in memory.
template <int T>
__device__ void block_pick(SelState& st, const uint32_t* __restrict__ hist, int digit, uint32_t* part,
                           uint32_t* __restrict__ err) {
  constexpr int BPT = kHistBins / T;
  const int t = threadIdx.x;
  const int nbins = (int)digit_mask(digit) + 1;
  uint32_t h[BPT];
  static_assert(BPT % 4 == 0, "whole uint4 groups per thread");
#pragma unroll
  for (int j = 0; j < BPT / 4; ++j) {
    uint4 q = make_uint4(0u, 0u, 0u, 0u);
    if (BPT * t < nbins) q = reinterpret_cast<const uint4*>(hist)[(BPT / 4) * t + j];  // (nbins is a multiple of BPT)
    h[4 * j + 0] = q.x;
    h[4 * j + 1] = q.y;
    h[4 * j + 2] = q.z;
    h[4 * j + 3] = q.w;
  }
  block_pick_bins<T>(st, h, digit, part, err);
}

// State at `want_level` (2 or 3) in st (shared).  st.compact_level = the level
// whose pass writes the survivor list (1, 2 or 3), st.list_count its size.
template <int T>
__device__ void derive_state(const SegView& sv, SelState& st, int want_level, uint32_t* part,
                             uint32_t* __restrict__ err) {
  if (threadIdx.x == 0) st = *sv.st;  // level 1; compact_level = 1 if the level-1 survivors fit
  __syncthreads();
  block_pick<T>(st, sv.hist1, 1, part, err);
  if (threadIdx.x == 0 && st.compact_level == 0u) {
    if (fits_list(st, sv.d.cap)) {
      st.compact_level = 2u;
      st.list_count = st.n_gt + st.cand;
    } else {
      st.compact_level = 3u;
    }
  }
  __syncthreads();
  if (want_level >= 3) {
    block_pick<T>(st, sv.hist2, 2, part, err);
    if (threadIdx.x == 0 && st.compact_level == 3u) st.list_count = st.n_gt + (st.cand < st.need ? st.cand : st.need);
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// k_pick0 : one block of 1024 threads per segment.  Optionally first finishes
// the per-worker variances and takes the leader (flat VAR step).  Then: suffix
// sums of the top-digit histogram, threshold digit b0 = the largest b with at
// least k keys at or above it, the level-1 state, and for every chunk of the
// segment the offset of its survivors (keys with top digit >= b0) in the list.
// ---------------------------------------------------------------------------
struct LeaderArgs {
  const double* partials;  // nullptr: the leader is already in leader_dev
  int w_count, nblk;
  int64_t n;
  double* var_scratch;
  double* var_out;
  int32_t* leader_dev;
  int32_t* leader_out;
};

// Finishes the per-worker variances from the fused pass' partials and takes the first
// worker of largest variance (same arithmetic as k_leader).  All threads of the
// block call it; returns the leader in thread 0 only.
__device__ int block_take_leader(const LeaderArgs& la) {
  const int t = threadIdx.x;
  const int wave = t >> 6, lane = t & 63;
  for (int w = wave; w < la.w_count; w += (int)blockDim.x / 64) {
    const double v = wave_variance(la.partials, w, la.nblk);
    if (lane == 0) {
      la.var_scratch[w] = v;
      if (la.var_out) la.var_out[w] = v;
    }
  }
  __threadfence_block();
  __syncthreads();
  int best = 0;
  if (t == 0) {
    for (int w = 1; w < la.w_count; ++w)
      if (la.var_scratch[w] > la.var_scratch[best]) best = w;
    *la.leader_dev = best;
    if (la.leader_out) *la.leader_out = best;
  }
  return best;
}

__device__ __forceinline__ void pick0_body(const SelParams& p, const LeaderArgs& la, int seg, uint32_t* part) {
  __shared__ int b0_sh;
  __shared__ int lead_sh;
  const int t = threadIdx.x;
  if (t == 0) {
    b0_sh = -1;
    lead_sh = -1;
  }
  if (la.partials != nullptr) {
    const int best = block_take_leader(la);
    if (t == 0) lead_sh = best;
  }
  __syncthreads();
  const SegView sv = seg_view(p, seg, lead_sh);
  if (p.only_if_need_full && sv.st->need_full == 0u) return;
  if (p.from_list && sv.st->use_mask == 0u) return;
  const SelState prev = *sv.st;  // from_list: says how long the list is
  bool from_list = p.from_list != 0;
  const uint32_t* __restrict__ htop = sv.htop;
  int htop_reps = sv.htop_reps;
  if (p.after_mask) {  // the list was written from the mask, or k_hist0's work has just been done instead
    if (prev.use_mask != 0u) {
      from_list = true;
    } else if (prev.need_full != 0u) {
      htop = sv.hseg;
      htop_reps = 1;
    } else {
      return;
    }
  }
  const uint32_t k = sv.d.k;
  const int nchunks = sv.d.geom.nchunks;

  // suffix sums of the top-digit histogram: sx[j] = keys with digit >= 4t+j
  uint32_t h[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) h[j] = 0u;
  for (int r0 = 0; r0 < htop_reps; r0 += 8) {  // eight loads in flight together (one copy: the same one, used once)
    uint4 q[8];
#pragma unroll
    for (int r = 0; r < 8; ++r)
      q[r] = reinterpret_cast<const uint4*>(htop + (size_t)(r0 + r < htop_reps ? r0 + r : r0) * kHistBins)[t];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      if (r0 + r < htop_reps) {
        h[0] += q[r].x;
        h[1] += q[r].y;
        h[2] += q[r].z;
        h[3] += q[r].w;
      }
    }
  }
  const uint32_t hsum = h[0] + h[1] + h[2] + h[3];
  uint32_t sx[5];
  sx[4] = block_suffix_incl<1024>(hsum, part) - hsum;
#pragma unroll
  for (int j = 3; j >= 0; --j) sx[j] = sx[j + 1] + h[j];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (sx[j] >= k && sx[j + 1] < k) {  // the suffix sums are non-increasing: one hit
      b0_sh = 4 * t + j;
      SelState st{};
      st.lo = (uint32_t)(4 * t + j) << 19;
      st.hi = st.lo | 0x7ffffu;
      st.n_gt = sx[j + 1];
      st.need = k - sx[j + 1];
      st.cand = sx[j] - sx[j + 1];
      st.level = 1u;
      if (from_list) {  // the list exists already and holds every key >= list_lo
        st.compact_level = 1u;
        st.use_mask = 1u;
        st.list_lo = prev.list_lo;
        st.list_count = prev.list_count;
      } else {
        st.compact_level = fits_list(st, sv.d.cap) ? 1u : 0u;
        st.list_count = st.compact_level ? st.n_gt + st.cand : 0u;
      }
      *sv.st = st;
    }
  }
  __syncthreads();
  const int b0 = b0_sh;
  if (b0 < 0) {
    if (t == 0) atomicOr(p.err, kErrPick);
    return;
  }
  if (from_list) return;
  // exclusive scan of the per-chunk survivor counts
  const uint32_t mine = (t < nchunks) ? sv.S[(size_t)t * kHistBins + b0] : 0u;
  const uint32_t upto = block_prefix_incl<1024>(mine, part);
  if (t < nchunks) sv.chunk_off[t] = upto - mine;
}

__global__ void __launch_bounds__(1024)
k_pick0(SelParams p, LeaderArgs la) {
  __shared__ uint32_t part[1024];
  pick0_body(p, la, blockIdx.y, part);
}

// ---------------------------------------------------------------------------
// k_pick_mask : first selection kernel after a fused pass that marked the keys
// reaching a guessed bound.  One block of 1024 threads (flat selections only).
// Optionally takes the leader first.  Adds up the per-chunk counts of marked
// elements; if the bound holds at least k and at most min(cap, k + n/8) keys, every
// marked element will become a list entry (chunk offsets are written, the state stays
// at level 0 with use_mask set); otherwise the state asks for the histogram of
// every key (need_full).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(1024)
k_pick_mask(SelParams p, LeaderArgs la) {
  __shared__ uint32_t part[1024];
  __shared__ int lead_sh;
  const int t = threadIdx.x;
  if (t == 0) lead_sh = -1;
  if (la.partials != nullptr) {
    const int best = block_take_leader(la);
    if (t == 0) lead_sh = best;
  }
  __syncthreads();
  const SegView sv = seg_view(p, blockIdx.y, lead_sh);
  const uint32_t k = sv.d.k;
  const int nchunks = sv.d.geom.nchunks;
  const uint32_t gkey = sv.ctrl[1];
  const uint32_t mine = (t < nchunks) ? sv.mcount[t * kMcountLine] : 0u;
  uint32_t total;
  const uint32_t upto = block_prefix_incl<1024>(mine, part, &total);
  // accepted if the bound holds at least k keys and not more than the list takes; a list far
  // longer than k (beyond k + n/8) is not worth fetching entry by entry either
  const uint64_t span = (uint64_t)(sv.d.e_hi - sv.d.e_lo);
  uint64_t limit = (uint64_t)k + (span >> 3);
  if (limit > sv.d.cap) limit = sv.d.cap;
  const bool ok = gkey != kNoGuess && total >= k && total <= limit;
  if (ok && t < nchunks) sv.chunk_off[t] = upto - mine;
  if (t == 0) {
    SelState st{};
    if (ok) {
      st.hi = kKeyMask;
      st.need = k;
      st.cand = total;
      st.compact_level = 1u;
      st.use_mask = 1u;
      st.list_lo = gkey;
      st.list_count = total;
    } else {
      st.need_full = 1u;
    }
    *sv.st = st;
  }
}

// ---------------------------------------------------------------------------
// k_compact1 : level-1 compaction of the leader's range, one block per chunk.
// Survivors (key >= st.lo, i.e. top digit >= b0) are written to the survivor
// list in ascending element order at chunk_off[c] + rank inside the chunk;
// candidates (top digit == b0) also feed the next-digit histogram hist1.
// If the list cannot hold n_gt + cand entries nothing is written and only the
// histogram is built.  block = WAVES waves; in a tile every lane owns 4 R
// consecutive elements (lane-contiguous loads run at the same bandwidth as
// row-coalesced ones here), so a survivor's rank is the lane's exclusive prefix
// plus its position among the lane's own survivors: five or six ballots per
// tile instead of one per element.
//   Bound by instructions issued, not by memory: with the survivors handled where
// they are found (sixteen predicated blocks a lane, run by every wave as soon as one of
// its lanes has any) the kernel took 152 us on 138 M elements and 42 on 25.6 M in 54
// segments.  Now a lane only lists its survivors' places on chip and the wave then
// takes them one per lane, values from the tile's on-chip copy: 141 and 34.5 us.
// Shapes (138 M select, whole call): 8 waves x 16 elements 303 us, 8 x 8 325, 4 x 16
// 333, 16 x 16 310, 16 x 8 328.
//   Tiles in which more than a quarter survives, and survivors that are only counted, go from
// the registers as before (60 M equal values 229 us, staged 295; an eighth or a half for a
// quarter: the same), so that the stage needs places for a quarter of a tile: 54 instead of
// 66 KB a block of 8 waves, 35 instead of 58 in k_level1 with 4, whose two jobs share one
// histogram.  Tiles in which all survive need no places and are staged (registers / staged
// with places / without, us: 3 M of one top digit 29/18/17, of two values 27/23/19; one in ten
// of 11.7 M sorted ones, all the work in a few blocks, 30/40/34).
// ---------------------------------------------------------------------------
constexpr int kC1Waves = 4, kC1R = 4;  // (flat vectors on the histogram route take 8 waves)

// lh: kHistBins words on chip.
template <int WAVES, int R>
__device__ __forceinline__ void compact1_body(const SelParams& p, uint32_t* __restrict__ lh) {
  constexpr int T = 64 * WAVES;
  constexpr int E = 4 * R;             // consecutive elements one lane owns in a tile (a power of two)
  constexpr int WSPAN = 64 * E;        // consecutive elements one wave owns in a tile
  constexpr int TILE = WAVES * WSPAN;  // elements per block iteration
  constexpr int FEW = WSPAN / 4;       // survivors of a wave's tile that are taken one per lane
  static_assert(E <= 32, "one 32-bit mask per lane");
  __shared__ uint32_t wtot[2][WAVES];
  __shared__ __attribute__((aligned(16))) uint32_t tile_raw[WAVES][WSPAN];  // a wave's tile, group r of lane l at 256 r + 4 l
  __shared__ uint16_t tile_pos[WAVES][FEW];                                 // its survivors' places in the wave's tile

  int seg, c;
  block_chunk(p, seg, c);
  const SegView sv = seg_view(p, seg);
  if (c >= sv.d.geom.nchunks) return;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t lane = lane_id();
  const int64_t n = p.n, e_lo = sv.d.e_lo, e_hi = sv.d.e_hi;
  const ChunkGeom geom = sv.d.geom;
  const uint32_t cap = sv.d.cap;
  uint2* __restrict__ list = sv.list;

  const SelState st = *sv.st;
  if (st.level != 1u || st.use_mask != 0u || *p.err) return;
  const bool write_out = st.compact_level == 1u;  // the level-1 survivors fit the list
  const bool zero_out = write_out && p.zero_vec != nullptr;
  const uint32_t klo = st.lo, khi = st.hi;
  const float* __restrict__ xp = sv.x;

  for (int b = tid; b < kHistBins; b += T) lh[b] = 0u;
  __syncthreads();

  const int64_t c_begin = geom.chunk0 + (int64_t)c * geom.chunk_elems;  // a multiple of kTile
  const int64_t c_end = c_begin + geom.chunk_elems;
  const int64_t cs = c_begin > e_lo ? c_begin : e_lo;  // elements of the range owned by this chunk
  const int64_t ce = c_end < e_hi ? c_end : e_hi;
  const int64_t n_vec = n & ~(int64_t)3;
  const int64_t lane_off = (int64_t)wave * WSPAN + (int64_t)lane * E;

  uint32_t run = write_out ? sv.chunk_off[c] : 0u;  // list position of the next survivor of this chunk
  int buf = 0;

  // raw bits of one tile; a tile that is wholly inside the array is read with R unconditional loads
  // (conditions around the loads make the compiler wait for each before issuing the next), in the
  // last tile groups are read element by element where needed, absent elements as 0
  auto load_tile = [&](int64_t tb, uint32_t (&out)[E]) {
    const int64_t j0 = tb + lane_off;
    if (tb + TILE <= n_vec) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const uint4 v = *reinterpret_cast<const uint4*>(xp + j0 + 4 * r);
        out[4 * r + 0] = v.x;
        out[4 * r + 1] = v.y;
        out[4 * r + 2] = v.z;
        out[4 * r + 3] = v.w;
      }
    } else {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int64_t j = j0 + 4 * r;
        uint4 v;
        if (j + 4 <= n_vec) {
          v = *reinterpret_cast<const uint4*>(xp + j);
        } else {
          v.x = (j + 0 < n) ? __float_as_uint(xp[j + 0]) : 0u;
          v.y = (j + 1 < n) ? __float_as_uint(xp[j + 1]) : 0u;
          v.z = (j + 2 < n) ? __float_as_uint(xp[j + 2]) : 0u;
          v.w = (j + 3 < n) ? __float_as_uint(xp[j + 3]) : 0u;
        }
        out[4 * r + 0] = v.x;
        out[4 * r + 1] = v.y;
        out[4 * r + 2] = v.z;
        out[4 * r + 3] = v.w;
      }
    }
  };

  // the next tile's loads are issued before this tile is worked on
  uint32_t raw[E], nxt[E];
  if (c_begin < ce) load_tile(c_begin, raw);
  for (int64_t tb = c_begin; tb < ce; tb += TILE) {
    const int64_t j0 = tb + lane_off;  // this lane's E consecutive elements start here
    const bool more = tb + TILE < ce;
    if (more) load_tile(tb + TILE, nxt);
    // every element of this tile belongs to the chunk and the range?
    const bool clean = (tb >= cs) && (tb + TILE <= ce);

    // survivors (key >= klo) among this lane's elements, one bit each
    uint32_t own = 0u;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      bool ok = (raw[e] & kKeyMask) >= klo;
      if (!clean) ok = ok && (j0 + e >= cs) && (j0 + e < ce);
      own |= ok ? (1u << e) : 0u;
    }
    const uint32_t cnt = (uint32_t)__popc(own);
    // exclusive prefix of cnt over the lanes and the wave total, from the bit planes of cnt
    uint32_t before = 0u, wsum = 0u;
#pragma unroll
    for (int b = 0; (1 << b) <= E; ++b) {
      const uint64_t plane = __ballot((cnt >> b) & 1u);
      before += popc_lt(plane) << b;
      wsum += (uint32_t)__popcll(plane) << b;
    }

    uint32_t base = 0u;
    if (write_out) {
      if (lane == 0) wtot[buf][wave] = wsum;
      __syncthreads();
      base = run;
#pragma unroll
      for (int i = 0; i < WAVES; ++i) {
        const uint32_t wt = wtot[buf][i];
        if (i < wave) base += wt;
        run += wt;
      }
      buf ^= 1;
    }
    const bool full = wsum == (uint32_t)WSPAN;  // every element of the wave's tile
    if ((wsum > (uint32_t)FEW && !full) || !write_out) {  // many, or only to be counted: from the registers
      uint32_t pos = base + before;
#pragma unroll
      for (int e = 0; e < E; ++e) {
        if ((own >> e) & 1u) {
          const uint32_t kk = raw[e] & kKeyMask;
          if (kk <= khi)
            atomicAdd(&lh[(kk >> 7) & 0xfffu], 1u);
          else if (zero_out)
            p.zero_vec[j0 + e] = 0.0f;
          if (write_out && pos < cap) list[pos] = make_uint2((uint32_t)(j0 + e), raw[e]);
          ++pos;
        }
      }
    } else if (wsum != 0u) {
      uint32_t* __restrict__ traw = tile_raw[wave];
      uint16_t* __restrict__ tpos = tile_pos[wave];
#pragma unroll
      for (int r = 0; r < R; ++r)
        reinterpret_cast<uint4*>(traw)[r * 64 + lane] =
            make_uint4(raw[4 * r + 0], raw[4 * r + 1], raw[4 * r + 2], raw[4 * r + 3]);
      // every lane lists its survivors; few lanes have more than one or two
      uint32_t pos = before;
      for (uint32_t left = full ? 0u : own; left != 0u; left &= left - 1u) {
        tpos[pos] = (uint16_t)(lane * E + (uint32_t)__builtin_ctz(left));
        ++pos;
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      // then the wave takes them one per lane: list entries go out side by side
      for (uint32_t i = lane; i < wsum; i += 64u) {
        const uint32_t q = full ? i : tpos[i];  // element q of the wave's tile: lane q / E, group (q / 4) mod R
        const uint32_t w = traw[((q >> 2) & (uint32_t)(R - 1)) * 256u + (q / E) * 4u + (q & 3u)];
        const uint32_t kk = w & kKeyMask;
        const uint32_t j = (uint32_t)(tb + (int64_t)wave * WSPAN) + q;
        // (index, raw bits): the sign travels with the survivor
        if (base + i < cap) list[base + i] = make_uint2(j, w);
        if (kk <= khi)
          atomicAdd(&lh[(kk >> 7) & 0xfffu], 1u);  // candidate: feeds the next digit
        else if (zero_out)
          // Keys above the threshold digit are kept whatever the later digits say: if asked to, put
          // +0.0 there now (the list carries the values on).  Only when the list is written here,
          // because the deeper array passes would re-read the vector.
          p.zero_vec[j] = 0.0f;
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();  // (the next tile overwrites the wave's stage)
    }
    if (more) {
#pragma unroll
      for (int e = 0; e < E; ++e) raw[e] = nxt[e];
    }
  }

  __syncthreads();
  for (int b = tid; b < kHistBins; b += T) {
    const uint32_t v = lh[b];
    if (v) atomicAdd(&sv.hist1[b], v);
  }
}

// ---------------------------------------------------------------------------
// compact_mask_body (first job of k_mask_or_hist) : writes the survivor list from the
// bit mask the fused pass left behind instead of re-reading the vector; one block of
// 1024 threads per chunk, runs only if the state says use_mask.  Every marked element (key >=
// list_lo) becomes a list entry, in ascending element order, starting at
// chunk_off[c]; only the marked elements' values are fetched.  The top digits
// of all entries are counted into the slot's partial whole-vector histograms
// (copy c mod kHistReps), from which k_pick0 then takes the threshold digit.
//   Per slab of 1024 mask rows (256 elements each), two steps.  First thread t
//   owns row t: a block scan of the rows' popcounts gives the row's list
//   offset, and the thread writes the indices of its marked elements into the
//   list entries.  Then the block walks the slab's entries with one entry per
//   thread, UB of them in flight, fetching the values to complete the entries.
// ---------------------------------------------------------------------------
template <int UB>
__device__ __forceinline__ void compact_mask_body(const SelParams& p) {
  constexpr int T = 1024, WAVES = 16;
  constexpr uint32_t STAGE = 4096;  // a slab with at most this many marks keeps their indices on chip
  __shared__ uint32_t wtot[WAVES];
  __shared__ uint32_t lh[kHistBins];
  __shared__ uint32_t sidx[STAGE];

  const SegView sv = seg_view(p, blockIdx.y);
  const int c = blockIdx.x;
  if (c >= sv.d.geom.nchunks) return;
  const SelState st = *sv.st;
  if (st.use_mask == 0u || sv.mask == nullptr || *p.err) return;
  const int tid = threadIdx.x;
  const int wave = tid >> 6;
  const uint32_t lane = lane_id();
  const int64_t n = p.n;
  const ChunkGeom geom = sv.d.geom;
  const uint32_t cap = sv.d.cap;
  const uint32_t list_lo = st.list_lo;
  const float* __restrict__ xp = sv.x;
  const uint64_t* __restrict__ mk = sv.mask;
  uint2* list = sv.list;

  for (int b = tid; b < kHistBins; b += T) lh[b] = 0u;
  __syncthreads();

  const int64_t c_begin = geom.chunk0 + (int64_t)c * geom.chunk_elems;  // a multiple of 256
  int64_t c_end = c_begin + geom.chunk_elems;
  if (c_end > n) c_end = n;
  const int64_t n_vec = n & ~(int64_t)3;                      // marked elements end here
  const int64_t v_end = c_end < n_vec ? c_end : n_vec;
  const int64_t row_lo = c_begin >> 8;
  const int64_t row_hi = (v_end + 255) >> 8;                  // exclusive

  uint32_t run = sv.chunk_off[c];  // list position of the next entry of this chunk
  // a row's four mask words; rows behind the chunk re-read its last row (unused), so that the
  // loads sit in no branch and the next slab's can be in flight while this slab is worked on
  auto load_row = [&](int64_t row, uint4& lo2, uint4& hi2) {
    const int64_t rr = row < row_hi ? row : row_hi - 1;
    lo2 = reinterpret_cast<const uint4*>(mk + mask_word(rr))[0];
    hi2 = reinterpret_cast<const uint4*>(mk + mask_word(rr))[1];
  };
  uint4 cur_lo = make_uint4(0u, 0u, 0u, 0u), cur_hi = cur_lo;
  if (row_lo < row_hi) load_row(row_lo + tid, cur_lo, cur_hi);
  for (int64_t slab = row_lo; slab < row_hi; slab += T) {
    const int64_t row = slab + tid;
    uint4 nxt_lo = cur_lo, nxt_hi = cur_hi;
    if (slab + T < row_hi) load_row(row + T, nxt_lo, nxt_hi);  // block-uniform condition
    uint64_t m[4] = {0ull, 0ull, 0ull, 0ull};
    if (row < row_hi) {
      m[0] = ((uint64_t)cur_lo.y << 32) | cur_lo.x;
      m[1] = ((uint64_t)cur_lo.w << 32) | cur_lo.z;
      m[2] = ((uint64_t)cur_hi.y << 32) | cur_hi.x;
      m[3] = ((uint64_t)cur_hi.w << 32) | cur_hi.z;
    }
    const uint32_t cnt = (uint32_t)(__popcll(m[0]) + __popcll(m[1]) + __popcll(m[2]) + __popcll(m[3]));
    // exclusive prefix of cnt (<= 256) over the lanes and the wave total, from the bit planes of cnt
    uint32_t before = 0u, wsum = 0u;
#pragma unroll
    for (int b = 0; b <= 8; ++b) {
      const uint64_t plane = __ballot((cnt >> b) & 1u);
      before += popc_lt(plane) << b;
      wsum += (uint32_t)__popcll(plane) << b;
    }
    if (lane == 0) wtot[wave] = wsum;
    __syncthreads();
    uint32_t pos = run + before, total = 0u;
#pragma unroll
    for (int i = 0; i < WAVES; ++i) {
      const uint32_t wt = wtot[i];
      if (i < wave) pos += wt;
      total += wt;
    }
    // the row's marked elements in ascending order: by group, then by position in the group;
    // their indices go to the on-chip stage if the slab's marks fit there, else into the list
    const bool staged = total <= STAGE;  // the same in every thread
    uint64_t any = m[0] | m[1] | m[2] | m[3];
    while (any) {
      const int g = __builtin_ctzll(any);
      const uint64_t bit = 1ull << g;
      any &= ~bit;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (m[e] & bit) {
          const uint32_t j = (uint32_t)(row * 256 + 4 * g + e);
          if (staged)
            sidx[pos - run] = j;
          else if (pos < cap)
            list[pos].x = j;
          ++pos;
        }
      }
    }
    __threadfence_block();  // the indices are written before any thread of the block reads them
    __syncthreads();
    for (uint32_t e0 = (uint32_t)tid; e0 < total; e0 += T * UB) {
      uint32_t j[UB], raw[UB];
      bool ok[UB];
#pragma unroll
      for (int u = 0; u < UB; ++u) {
        const uint32_t e = e0 + (uint32_t)u * T;
        ok[u] = e < total && run + e < cap;
        j[u] = !ok[u] ? 0u : staged ? sidx[e] : list[run + e].x;
      }
#pragma unroll
      for (int u = 0; u < UB; ++u) raw[u] = __float_as_uint(xp[j[u]]);
#pragma unroll
      for (int u = 0; u < UB; ++u) {
        if (ok[u]) {
          if (staged)
            list[run + e0 + (uint32_t)u * T] = make_uint2(j[u], raw[u]);  // the whole entry at once
          else
            list[run + e0 + (uint32_t)u * T].y = raw[u];
          atomicAdd(&lh[(raw[u] & kKeyMask) >> 19], 1u);
        }
      }
    }
    run += total;
    cur_lo = nxt_lo;  // (only here: the copy waits for the loads)
    cur_hi = nxt_hi;
  }
  // the elements behind the last whole group of four are not in the mask
  if (c_end == n && n_vec < n && tid == 0) {
    for (int64_t j = n_vec; j < n; ++j) {
      const uint32_t raw = __float_as_uint(xp[j]);
      const uint32_t kk = raw & kKeyMask;
      if (kk >= list_lo) {
        atomicAdd(&lh[kk >> 19], 1u);
        if (run < cap) list[run] = make_uint2((uint32_t)j, raw);
        ++run;
      }
    }
  }

  __syncthreads();
  uint32_t* __restrict__ htop = sv.htop + (size_t)(c % sv.htop_reps) * kHistBins;
  for (int b = tid; b < kHistBins; b += T) {
    const uint32_t v = lh[b];
    if (v) atomicAdd(&htop[b], v);
  }
}

// ---------------------------------------------------------------------------
// Marking on vectors that are only read (k_mark_spans): a wave works alone on spans of
// 2048 or 8192 consecutive elements.  Per row of 64 float4 groups it needs the largest
// magnitude of each group, one comparison with the bound and, where a group reaches it,
// the group's place in a queue on chip; 64 queued groups at a time are then taken one per
// lane, their marked elements ranked (three ballots) and stored.  About 200 instructions a
// wave and 2048 elements, so that the stream of loads is what bounds it: 102 us on 138 M
// elements (5.4 TB/s), one in a hundred kept; a form of k_pass_mark that only read, about
// 1700 instructions, took 191, and the two passes of the histogram route take 116 + 141.
// ---------------------------------------------------------------------------
constexpr int kSpanStep = 2048;  // elements a wave loads at a time: 8 rows of 64 float4 groups
struct SpanQueue {
  uint4 val[128];      // the queued groups' raw bits
  uint32_t group[128]; // their numbers (element / 4)
};

// The elements of x[e0, min(e0 + span, n)) whose key reaches the bound, as (index, raw bits) in
// ascending order to dst[0 .. cap); returns their number, which may be larger than cap.  With lh their
// top digits are counted there.  The 64 lanes of a wave call it; gf is the bound as a float (an element
// is marked if not |x| < gf, so a NaN is).
template <bool NT>
__device__ __forceinline__ uint32_t wave_span(const float* __restrict__ x, int64_t n, int64_t e0, int span, float gf,
                                              SpanQueue& qu, uint2* __restrict__ dst, uint32_t cap,
                                              uint32_t* __restrict__ lh) {
  const uint32_t lane = lane_id();
  uint32_t count = 0u, head = 0u, queued = 0u;
  // takes the first m queued groups, one per lane
  auto take = [&](uint32_t m) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const uint32_t p = (head + lane) & 127u;
    const uint4 v = qu.val[p];
    const uint32_t g = qu.group[p];
    const uint32_t raw[4] = {v.x, v.y, v.z, v.w};
    uint32_t own = 0u;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      own |= (!(__builtin_fabsf(__uint_as_float(raw[e])) < gf) && (int64_t)4 * g + e < n) ? 1u << e : 0u;
    if (lane >= m) own = 0u;
    const uint32_t c = (uint32_t)__popc(own);
    uint32_t before = 0u, total = 0u;
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const uint64_t plane = __ballot((c >> b) & 1u);
      before += popc_lt(plane) << b;
      total += (uint32_t)__popcll(plane) << b;
    }
    uint32_t pos = count + before;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if ((own >> e) & 1u) {
        if (pos < cap) dst[pos] = make_uint2(4u * g + (uint32_t)e, raw[e]);
        if (lh != nullptr) atomicAdd(&lh[(raw[e] & kKeyMask) >> 19], 1u);
        ++pos;
      }
    }
    count += total;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();  // (what is queued next may overwrite these)
  };
  for (int64_t base = e0; base < e0 + span && base < n; base += kSpanStep) {
    const uint32_t g0 = (uint32_t)(base >> 2) + lane;
    v4f v[8];
    if (base + kSpanStep <= n) {
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = load4<NT>(x + 4 * (int64_t)(g0 + 64u * u));
    } else {  // the vector's end: absent elements as 0, which only a bound of 0 marks (take() looks again)
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int64_t j = 4 * (int64_t)(g0 + 64u * u);
        v[u] = v4f{0.f, 0.f, 0.f, 0.f};
        if (j + 4 <= n) {
          v[u] = load4<false>(x + j);
        } else {
          if (j + 0 < n) v[u].x = x[j + 0];
          if (j + 1 < n) v[u].y = x[j + 1];
          if (j + 2 < n) v[u].z = x[j + 2];
        }
      }
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const float top = __builtin_elementwise_maximum(
          __builtin_elementwise_maximum(__builtin_fabsf(v[u].x), __builtin_fabsf(v[u].y)),
          __builtin_elementwise_maximum(__builtin_fabsf(v[u].z), __builtin_fabsf(v[u].w)));  // NaN if any is
      const bool hit = !(top < gf);
      const uint64_t hits = __ballot(hit);
      if (hits != 0ull) {
        if (hit) {
          const uint32_t p = (head + queued + popc_lt(hits)) & 127u;
          qu.val[p] = make_uint4(__float_as_uint(v[u].x), __float_as_uint(v[u].y), __float_as_uint(v[u].z),
                                 __float_as_uint(v[u].w));
          qu.group[p] = g0 + 64u * u;
        }
        queued += (uint32_t)__popcll(hits);
        if (queued >= 64u) {
          take(64u);
          head += 64u;
          queued -= 64u;
        }
      }
    }
  }
  if (queued != 0u) take(queued);
  return count;
}

// grid = (blocks, vectors), block = 256; vector y uses slot y and piece row y.  Every span's entries go to
// its piece, the first tiles.cap of them, and their number to tiles.cnt; a vector without a bound is left alone.
template <bool NT>
__global__ void __launch_bounds__(256)
k_mark_spans(PtrTable x, int64_t n, int64_t chunk_elems, uint32_t* __restrict__ h_all, TileBuf tiles) {
  __shared__ SpanQueue qu[4];
  const int v = blockIdx.y;
  uint32_t* __restrict__ slot = h_all + (size_t)v * kSlotWords;
  const uint32_t gkey = slot[kSlotCtrl + 1];
  if (gkey == kNoGuess) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t nspans = (n + tiles.span - 1) / tiles.span;
  uint2* __restrict__ buf = tiles.buf + (size_t)v * (size_t)tiles.buf_stride;
  uint32_t* __restrict__ cnt = tiles.cnt + (size_t)v * (size_t)tiles.cnt_stride;
  for (int64_t sp = (int64_t)blockIdx.x * 4 + wave; sp < nspans; sp += (int64_t)gridDim.x * 4) {
    const uint32_t c = wave_span<NT>(x.p[v], n, sp * tiles.span, tiles.span, __uint_as_float(gkey), qu[wave],
                                     buf + (size_t)sp * (size_t)tiles.cap, (uint32_t)tiles.cap, nullptr);
    if (lane_id() == 0) {
      cnt[sp] = c;
      if (c != 0u) atomicAdd(&slot[kSlotMcount + (sp * tiles.span) / chunk_elems * kMcountLine], c);
    }
  }
}

// The survivor list from the spans' pieces: one block of 1024 threads per chunk copies them, in order, to
// the list from chunk_off[c] on and counts the entries' top digits.  A span with more entries than its piece
// holds is marked again, into the list.
__device__ __forceinline__ void compact_spans_body(const SelParams& p) {
  constexpr int T = 1024, WAVES = T / 64;
  __shared__ uint32_t lh[kHistBins];
  __shared__ uint32_t pre[65];  // entries before each of 64 spans, and of all of them
  __shared__ SpanQueue qu[WAVES];

  const SegView sv = seg_view(p, blockIdx.y);
  const int c = blockIdx.x;
  if (c >= sv.d.geom.nchunks) return;
  const SelState st = *sv.st;
  if (st.use_mask == 0u || *p.err) return;
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int64_t n = p.n;
  const uint32_t cap = sv.d.cap, piece = (uint32_t)sv.tcap;
  const int64_t span = p.tiles.span;
  uint2* __restrict__ list = sv.list;

  for (int b = tid; b < kHistBins; b += T) lh[b] = 0u;
  const int64_t c_begin = sv.d.geom.chunk0 + (int64_t)c * sv.d.geom.chunk_elems;  // a whole number of spans
  int64_t c_end = c_begin + sv.d.geom.chunk_elems;
  if (c_end > n) c_end = n;
  const int64_t s_hi = (c_end + span - 1) / span;
  uint32_t run = sv.chunk_off[c];  // list position of the next entry of this chunk
  for (int64_t s0 = c_begin / span; s0 < s_hi; s0 += 64) {
    const int ns = (int)(s_hi - s0 < 64 ? s_hi - s0 : 64);
    const uint32_t mine = lane < ns ? sv.tcnt[s0 + lane] : 0u;  // (every wave scans the counts itself)
    const uint32_t incl = wave_incl_scan(mine);
    const uint32_t total = wave_last(incl);
    const uint64_t over = __ballot(mine > piece);
    __syncthreads();  // pre is free, and the histogram cleared
    if (wave == 0) {
      pre[lane] = incl - mine;
      if (lane == 63) pre[64] = total;
    }
    __syncthreads();
    for (uint32_t f0 = (uint32_t)tid; f0 < total; f0 += 2 * T) {
      uint2 ent[2];
      bool ok[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const uint32_t f = f0 + (uint32_t)u * T;
        const uint32_t fc = f < total ? f : total - 1u;
        int i = 0;  // the span this entry belongs to: the last whose first entry is not behind it
#pragma unroll
        for (int w = 32; w > 0; w >>= 1) i += pre[i + w] <= fc ? w : 0;
        const uint32_t r = fc - pre[i];
        ok[u] = f < total && r < piece && pre[i + 1] - pre[i] <= piece;
        ent[u] = sv.tbuf[(size_t)(s0 + i) * piece + (r < piece ? r : 0u)];
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const uint32_t f = f0 + (uint32_t)u * T;
        if (ok[u]) {
          if (run + f < cap) list[run + f] = ent[u];
          atomicAdd(&lh[(ent[u].y & kKeyMask) >> 19], 1u);
        }
      }
    }
    for (int i = wave; i < ns; i += WAVES) {
      if ((over >> i) & 1ull) {
        const uint32_t at = run + pre[i];
        wave_span<false>(sv.x, n, (s0 + i) * span, (int)span, __uint_as_float(st.list_lo), qu[wave], list + at,
                         at < cap ? cap - at : 0u, lh);
      }
    }
    run += total;
  }
  __syncthreads();
  uint32_t* __restrict__ htop = sv.htop + (size_t)(c % sv.htop_reps) * kHistBins;
  for (int b = tid; b < kHistBins; b += T) {
    const uint32_t v = lh[b];
    if (v) atomicAdd(&htop[b], v);
  }
}

// The kernel behind k_pick_mask where k_mark_spans left pieces: the list from them, or k_hist0's work.
__global__ void __launch_bounds__(1024)
k_spans_or_hist(SelParams p, SelParams p_full) {
  const SelState* st = seg_view(p, blockIdx.y).st;
  if (st->use_mask != 0u)
    compact_spans_body(p);
  else if (st->need_full != 0u)
    hist0_body<1024>(p_full);
}

// k_mask_or_hist : the kernel behind k_pick_mask.  Per segment it does whichever of the two
// jobs the state asks for: the list from the mask (use_mask), or, after a guess that did not
// hold, the per-chunk histograms of every key (need_full; p_full are the parameters of that
// route: own top-digit histogram, only_if_need_full set).  Both are one 1024-thread block per
// chunk, so they share a launch.
template <int UB>
__global__ void __launch_bounds__(1024)
k_mask_or_hist(SelParams p, SelParams p_full) {
  const SelState* st = seg_view(p, blockIdx.y).st;
  if (st->use_mask != 0u)
    compact_mask_body<UB>(p);
  else if (st->need_full != 0u)
    hist0_body<1024>(p_full);
}

// ---------------------------------------------------------------------------
// Decoupled look-back over tiles.  Each tile publishes a 64-bit word
//   [63:62] status (0 none, 1 tile aggregate, 2 inclusive prefix)
//   [61:31] count A (keys above the range)      [30:0] count B (keys inside)
// Counts never exceed 2^31-1 in total, so packed words add field-wise.
// Called by the 64 lanes of one wave; returns the exclusive prefix of `tile`.
// The wait on a predecessor is bounded; expiry sets *err and returns what was
// gathered so far (every wave still leaves the kernel).
// ---------------------------------------------------------------------------
constexpr uint64_t kFlagAgg = 1ull << 62;
constexpr uint64_t kFlagIncl = 2ull << 62;
constexpr uint64_t kFlagValMask = (1ull << 62) - 1ull;
constexpr int kSpinLimit = 1 << 20;

__device__ __forceinline__ uint64_t flag_load(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void flag_store(uint64_t* p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Flag word of a tile: `flags` + 0 or 1 for the array passes, the words behind those for the list pass.
template <bool LIST>
__device__ __forceinline__ uint64_t* flag_word(uint64_t* flags, int64_t tile) {
  return LIST ? flags + (tile >> 2) * kNumLookback + 2 + (tile & 3) : flags + tile * kNumLookback;
}

template <bool LIST>
__device__ uint64_t lookback_exclusive(uint64_t* __restrict__ flags, int64_t tile, uint64_t agg,
                                       uint32_t* __restrict__ err) {
  const uint32_t lane = lane_id();
  if (tile == 0) {
    if (lane == 0) flag_store(flag_word<LIST>(flags, 0), kFlagIncl | agg);
    return 0ull;
  }
  if (lane == 0) flag_store(flag_word<LIST>(flags, tile), kFlagAgg | agg);
  uint64_t excl = 0ull;     // wave-uniform running total
  int64_t base = tile - 1;  // lane L inspects tile base - L
  while (true) {
    const int64_t my = base - (int64_t)lane;
    uint64_t word = kFlagIncl;  // tiles before the first act as an inclusive prefix of zero
    if (my >= 0) {
      int spins = 0;
      word = flag_load(flag_word<LIST>(flags, my));
      while ((word >> 62) == 0ull) {
        if (++spins > kSpinLimit) {
          atomicOr(err, kErrWait);
          word = kFlagIncl;
          break;
        }
        __builtin_amdgcn_s_sleep(2);
        word = flag_load(flag_word<LIST>(flags, my));
      }
    }
    const uint64_t incl_mask = __ballot((word >> 62) == 2ull);
    uint64_t contrib = word & kFlagValMask;
    if (incl_mask != 0ull) {
      const int first = __ffsll((long long)incl_mask) - 1;  // nearest tile holding an inclusive prefix
      if ((int)lane > first) contrib = 0ull;
      excl += wave_allsum_u64(contrib);
      break;
    }
    excl += wave_allsum_u64(contrib);
    base -= 64;
  }
  if (lane == 0) flag_store(flag_word<LIST>(flags, tile), kFlagIncl | ((excl + agg) & kFlagValMask));
  return excl;
}

// ---------------------------------------------------------------------------
// k_compact : ordered compaction with two classes.
//   class A: key > st.hi           class B: st.lo <= key <= st.hi
//   An element is kept if it is in A, or in B with fewer than `quota` B
//   elements before it; its output position is
//        (#A before it) + min(#B before it, quota)
//   which is ascending in element order.  quota = infinity below level 3.
//
//   Elements are x[e_lo .. e_hi) of the selected vector, kept entries go to the
//   survivor list as (index, bits).  Level 2 runs when the level-1 survivors did
//   not fit the list, level 3 when the level-2 ones did not either; a pass writes
//   the list only if it fits (otherwise it only feeds the next digit histogram).
//   The pass over the list itself is list_final_body.
//
//   block = 512 threads = 8 waves; a tile is 8 waves x 8 rows x 64 lanes x 4
//   consecutive elements, each wave owning a contiguous 2048-element piece.
// ---------------------------------------------------------------------------
constexpr int kCompactThreads = 512;
constexpr int kCompactRows = 8;
constexpr int kCompactTile = kCompactThreads * 4 * kCompactRows;  // 16384 elements
constexpr int kWaveSpan = 64 * 4 * kCompactRows;                  // 2048 elements

// The pass itself; st is the state derived for it (in shared memory, the same in every thread).
// DIRECT (array source, level 3): the kept entries go straight to idx_out / vals_row (and are put
// to +0.0 in zero_vec) instead of into the list, so no pass over the list has to follow.
template <bool DIRECT>
__device__ __forceinline__ void compact_body(const SelParams& p, const SegView& sv, const SelState& st, int level,
                                             int launch_id, uint32_t zero_below) {
  __shared__ uint32_t lh[!DIRECT ? kHistBins : 4];
  __shared__ uint64_t wave_tot[8];
  __shared__ uint64_t tile_excl;
  __shared__ int64_t tile_sh;

  const int64_t n = p.n, e_lo = sv.d.e_lo, e_hi = sv.d.e_hi;
  const uint32_t cap = sv.d.cap;
  uint32_t* __restrict__ hist_next = sv.hist2;
  uint64_t* __restrict__ flags = sv.flags + launch_id;
  uint32_t* __restrict__ tile_counter = sv.counters + launch_id;
  uint2* __restrict__ list = sv.list;
  int32_t* __restrict__ idx_out = sv.idx_out;
  float* __restrict__ vals_row = sv.vals_row;
  const uint32_t k_out = sv.d.k;
  uint32_t* __restrict__ err = p.err;

  const int tid = threadIdx.x;
  const int wave = tid >> 6;
  const uint32_t lane = lane_id();

  // With zeroing on the way: the level-1 pass zeroed the keys above its range if it wrote the
  // list (zero_below = the top of that range); the pass that writes idx_out zeroes the kept rest,
  // or all of them otherwise (zero_below = every key).
  float* __restrict__ zero_vec = DIRECT ? p.zero_vec : nullptr;
  // level 2 runs whenever level 1 did not fit; level 3 only if level 2 did not fit either
  if (level == 3 && st.compact_level != 3u) return;
  const uint32_t quota = (level == 3) ? st.need : kQuotaInf;
  const bool write_out = st.compact_level == (uint32_t)level;
  const bool do_hist = level < 3 && !DIRECT;
  const int64_t first_tile = e_lo / kCompactTile;
  const int64_t ntiles = (e_hi + kCompactTile - 1) / kCompactTile - first_tile;
  const uint32_t klo = st.lo, khi = st.hi;
  const int dshift = digit_shift(level < 3 ? level : 2);
  const uint32_t dmask = digit_mask(level < 3 ? level : 2);

  const float* __restrict__ xp = sv.x;

  if (do_hist) {
    for (int b = tid; b < kHistBins; b += kCompactThreads) lh[b] = 0u;
  }
  __syncthreads();

  while (true) {
    if (tid == 0) tile_sh = (int64_t)atomicAdd(tile_counter, 1u);
    __syncthreads();
    const int64_t trel = tile_sh;
    if (trel >= ntiles) break;
    const int64_t tbase = (first_tile + trel) * kCompactTile + (int64_t)wave * kWaveSpan;

    // ---- load keys ------------------------------------------------------
    uint32_t key[kCompactRows][4];
    uint32_t valid = 0u;  // bit (r*4+e)
    const bool full = (tbase >= e_lo) && (tbase + kWaveSpan <= e_hi) && (tbase + kWaveSpan <= (n & ~(int64_t)3));
    if (full) {
#pragma unroll
      for (int r = 0; r < kCompactRows; ++r) {
        const int64_t j = tbase + (int64_t)r * 256 + (int64_t)lane * 4;
        const uint4 v = *reinterpret_cast<const uint4*>(xp + j);
        key[r][0] = v.x;  // raw bits; comparisons mask the sign off
        key[r][1] = v.y;
        key[r][2] = v.z;
        key[r][3] = v.w;
      }
      valid = 0xffffffffu;
    } else {
#pragma unroll
      for (int r = 0; r < kCompactRows; ++r) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int64_t j = tbase + (int64_t)r * 256 + (int64_t)lane * 4 + e;
          key[r][e] = 0u;
          if (j >= e_lo && j < e_hi) {
            valid |= 1u << (r * 4 + e);
            key[r][e] = __float_as_uint(xp[j]);
          }
        }
      }
    }

    // ---- classify, count, feed the next-digit histogram ----------------
    uint32_t isA = 0u, isB = 0u;
    uint32_t cntA = 0u, cntB = 0u;  // wave totals (uniform)
#pragma unroll
    for (int r = 0; r < kCompactRows; ++r) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool ok = (valid >> (r * 4 + e)) & 1u;
        const uint32_t mk = key[r][e] & kKeyMask;
        const bool a = ok && mk > khi;
        const bool b = ok && mk >= klo && mk <= khi;
        if (a) isA |= 1u << (r * 4 + e);
        if (b) isB |= 1u << (r * 4 + e);
        cntA += (uint32_t)__popcll(__ballot(a));
        cntB += (uint32_t)__popcll(__ballot(b));
        if (do_hist && b) atomicAdd(&lh[(mk >> dshift) & dmask], 1u);
      }
    }

    if (write_out) {
      if (lane == 0) wave_tot[wave] = ((uint64_t)cntA << 31) | (uint64_t)cntB;
      __syncthreads();
      if (wave == 0) {
        uint64_t agg = 0ull;
#pragma unroll
        for (int i = 0; i < 8; ++i) agg += wave_tot[i];
        const uint64_t ex = lookback_exclusive<false>(flags, trel, agg, err);
        if (lane == 0) tile_excl = ex;
      }
      __syncthreads();
      uint64_t mine = tile_excl;
      for (int i = 0; i < wave; ++i) mine += wave_tot[i];
      uint32_t runA = (uint32_t)(mine >> 31);
      uint32_t runB = (uint32_t)(mine & 0x7fffffffu);

      if ((cntA | cntB) != 0u) {
#pragma unroll
        for (int r = 0; r < kCompactRows; ++r) {
          uint64_t bA[4], bB[4];
          uint32_t rowA = 0u, rowB = 0u, ltA = 0u, ltB = 0u;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            bA[e] = __ballot((isA >> (r * 4 + e)) & 1u);
            bB[e] = __ballot((isB >> (r * 4 + e)) & 1u);
            rowA += (uint32_t)__popcll(bA[e]);
            rowB += (uint32_t)__popcll(bB[e]);
          }
          if ((rowA | rowB) != 0u) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              ltA += popc_lt(bA[e]);
              ltB += popc_lt(bB[e]);
            }
            uint32_t befA = runA + ltA, befB = runB + ltB;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const bool a = (isA >> (r * 4 + e)) & 1u;
              const bool b = (isB >> (r * 4 + e)) & 1u;
              if (a || (b && befB < quota)) {
                const uint32_t pos = befA + (befB < quota ? befB : quota);
                const int64_t j = tbase + (int64_t)r * 256 + (int64_t)lane * 4 + e;
                if (DIRECT) {
                  if (pos < k_out) {
                    idx_out[pos] = (int32_t)j;
                    if (vals_row) vals_row[pos] = __uint_as_float(key[r][e]);
                    if (zero_vec && ((key[r][e] & kKeyMask) <= zero_below) && j < p.n) zero_vec[j] = 0.0f;
                  }
                } else if (pos < cap) {
                  list[pos] = make_uint2((uint32_t)j, key[r][e]);
                }
              }
              befA += a ? 1u : 0u;
              befB += b ? 1u : 0u;
            }
          }
          runA += rowA;
          runB += rowB;
        }
      }
    }
    __syncthreads();  // tile_sh / wave_tot / tile_excl reused by the next tile
  }

  if (do_hist) {
    __syncthreads();
    for (int b = tid; b < kHistBins; b += kCompactThreads) {
      const uint32_t v = lh[b];
      if (v) atomicAdd(&hist_next[b], v);
    }
  }
}

// ---------------------------------------------------------------------------
// list_final_body : the final pass over the survivor list.  Kept entries (the two classes
// above, with the tie quota) go to idx_out[0 .. k) in list order, their values (the list
// carries the raw bits) to vals_row, and +0.0 to zero_vec where the key is <= zero_below.
//   Bound by its chain of dependent steps, not by bytes: lists are short (k entries and some),
// so tiles are small (512 threads of PER consecutive entries) to spread them over the chip; ranks
// come from the bit planes of the lanes' counts (eight or ten ballots a tile); the kept entries are
// collected on chip and stored side by side.  The form before it (16384 entries a tile, 128
// ballots, entries stored from where they are found) took 20 us on 12 thousand entries, 20 on
// 120 thousand, 22.5 on 1.4 million, 95 on 14.5 million; this one 9 / 11 / 26 / 105 with PER = 8
// and 12 / 13 / 19 / 92 with 16: the more tiles, the longer the walk back over their flags takes
// (more tiles per step of that walk, or more blocks at once, made it slower, not faster).
// Tiles come from a counter, so that a block never waits for one that has not started.
// ---------------------------------------------------------------------------
constexpr int kListTile = kCompactThreads * 8;  // the smallest tile: 4096 entries
static_assert(kCompactTile == 4 * kListTile, "four flag words of the list pass per array tile");

// Entries a lane takes of a list: 16 if the list, or all the lists of the launch together (of which at least the kept
// entries are known), are long.  8 against 16, us: one list of 255 k 10.6/13.8, 512 k 13.8/14.4, 770 k 15.4/15.5, 800 k
// all equal 13.6/14.6, 1 M 17.8/16.5, 1.5 M all equal 24/16, 3 M all equal 36/27, 14 M 105/90; 8 lists of 25 k 12.2/14,
// of 40 k 12.7/14.8, of 255 k 29/26; 9 of 154 k 25/20; 54 of 255 k together 15.2/14.4.  (32 entries: 3 M all equal 24,
// lists that are mostly kept 15 to 25 % slower.)
constexpr uint32_t kLongList = 3u << 18;
__device__ __forceinline__ bool long_list(uint32_t entries, uint32_t k_all) {
  return entries > kLongList || k_all > kLongList;
}

// stage: kCompactThreads * PER entries on chip.
template <int PER>
__device__ __forceinline__ void list_final_body(const SelParams& p, const SegView& sv, const SelState& st,
                                                uint32_t zero_below, int64_t tile, uint2* __restrict__ stage) {
  constexpr int T = kCompactThreads, WAVES = T / 64, TILE = T * PER;
  __shared__ uint64_t wave_tot[WAVES];
  __shared__ uint64_t tile_excl;
  __shared__ int64_t tile_sh;

  const int tid = threadIdx.x;
  const int wave = tid >> 6;
  const uint32_t lane = lane_id();
  uint64_t* __restrict__ flags = sv.flags;
  uint32_t* __restrict__ tile_counter = sv.counters + 2;
  const uint2* __restrict__ list = sv.list;
  int32_t* __restrict__ idx_out = sv.idx_out;
  float* __restrict__ vals_row = sv.vals_row;
  float* __restrict__ zero_vec = p.zero_vec;
  const uint32_t k_out = sv.d.k;
  uint32_t* __restrict__ err = p.err;
  if (st.level != 3u) {
    if (tid == 0 && blockIdx.x == 0) atomicOr(err, kErrSequence);
    return;
  }
  const uint32_t quota = st.need, klo = st.lo, khi = st.hi, count = st.list_count;
  const int64_t ntiles = ((int64_t)count + TILE - 1) / TILE;

  while (tile < ntiles) {
    const uint32_t q0 = (uint32_t)(tile * TILE) + (uint32_t)tid * PER;
    // (the list's memory goes on for a whole tile behind its last entry)
    uint32_t raw[PER], ind[PER];
#pragma unroll
    for (int i = 0; i < PER / 2; ++i) {
      const uint4 v = reinterpret_cast<const uint4*>(list + q0)[i];
      ind[2 * i] = v.x;
      raw[2 * i] = v.y;
      ind[2 * i + 1] = v.z;
      raw[2 * i + 1] = v.w;
    }
    uint32_t isA = 0u, isB = 0u;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const uint32_t kk = raw[e] & kKeyMask;
      const bool ok = q0 + (uint32_t)e < count;
      isA |= (ok && kk > khi) ? 1u << e : 0u;
      isB |= (ok && kk >= klo && kk <= khi) ? 1u << e : 0u;
    }
    const uint32_t cA = (uint32_t)__popc(isA), cB = (uint32_t)__popc(isB);
    uint32_t befA = 0u, befB = 0u, totA = 0u, totB = 0u;
#pragma unroll
    for (int b = 0; (1 << b) <= PER; ++b) {
      const uint64_t pa = __ballot((cA >> b) & 1u), pb = __ballot((cB >> b) & 1u);
      befA += popc_lt(pa) << b;
      befB += popc_lt(pb) << b;
      totA += (uint32_t)__popcll(pa) << b;
      totB += (uint32_t)__popcll(pb) << b;
    }
    if (lane == 0) wave_tot[wave] = ((uint64_t)totA << 31) | (uint64_t)totB;
    __syncthreads();
    if (wave == 0) {
      uint64_t agg = 0ull;
#pragma unroll
      for (int i = 0; i < WAVES; ++i) agg += wave_tot[i];
      const uint64_t ex = lookback_exclusive<true>(flags, tile, agg, err);
      if (lane == 0) {
        tile_excl = ex;
        tile_sh = (int64_t)atomicAdd(tile_counter, 1u);  // this block's next tile
      }
    }
    __syncthreads();
    const uint64_t before_tile = tile_excl;
    uint64_t mine = before_tile, total = before_tile;
#pragma unroll
    for (int i = 0; i < WAVES; ++i) {
      const uint64_t wt = wave_tot[i];
      if (i < wave) mine += wt;
      total += wt;
    }
    // first output position of the tile, and behind its last
    auto place = [&](uint64_t ab) {
      const uint32_t a = (uint32_t)(ab >> 31), b = (uint32_t)(ab & 0x7fffffffu);
      return a + (b < quota ? b : quota);
    };
    const uint32_t p0 = place(before_tile), p1 = place(total);
    befA += (uint32_t)(mine >> 31);
    befB += (uint32_t)(mine & 0x7fffffffu);
    if ((isA | isB) != 0u) {
#pragma unroll
      for (int e = 0; e < PER; ++e) {
        const bool a = (isA >> e) & 1u, b = (isB >> e) & 1u;
        if (a || (b && befB < quota)) stage[befA + (befB < quota ? befB : quota) - p0] = make_uint2(ind[e], raw[e]);
        befA += a ? 1u : 0u;
        befB += b ? 1u : 0u;
      }
    }
    const int64_t next = tile_sh;
    __syncthreads();
    for (uint32_t i = (uint32_t)tid; i < p1 - p0; i += T) {
      const uint2 ent = stage[i];
      if (p0 + i < k_out) {
        idx_out[p0 + i] = (int32_t)ent.x;
        if (vals_row) vals_row[p0 + i] = __uint_as_float(ent.y);
        // kept entries that nothing has put to +0.0 yet
        if (zero_vec && (ent.y & kKeyMask) <= zero_below && (int64_t)ent.x < p.n) zero_vec[ent.x] = 0.0f;
      }
    }
    tile = next;  // (the next tile writes wave_tot before its first barrier and the stage behind its second:
                  //  every thread has left both by then)
  }
}

// Keys the level-1 pass has already put to +0.0 in zero_vec lie above this one (every key if it
// has not zeroed any).
__device__ __forceinline__ uint32_t zeroed_above(const SelState* stp) {
  return (stp->compact_level == 1u && stp->use_mask == 0u) ? stp->hi : kKeyMask;
}

// The level-2 pass over the array (where the level-1 survivors did not fit the list).
__global__ void __launch_bounds__(kCompactThreads)
k_compact(SelParams p) {
  __shared__ SelState st;
  __shared__ uint32_t pick_part[kCompactThreads];
  const SegView sv = seg_view(p, blockIdx.y);
  // the level-1 survivors fitted the list: nothing to do
  if (sv.st->compact_level == 1u || *p.err) return;
  derive_state<kCompactThreads>(sv, st, 2, pick_part, p.err);
  compact_body<false>(p, sv, st, 2, 0, kKeyMask);
}

// ---------------------------------------------------------------------------
// k_final : the last selection kernel.  If a list was written (at level 1, from the mask,
// or by the level-2 pass) it is the final pass over the list; if not even the level-2
// survivors fitted one (e.g. an all-equal vector) it is the level-3 pass over the array,
// which then writes the outputs itself.  ALWAYS_LIST: the list takes the whole vector, so
// the array passes do not exist.
// ---------------------------------------------------------------------------
template <bool ALWAYS_LIST>
__global__ void __launch_bounds__(kCompactThreads)
k_final(SelParams p) {
  __shared__ SelState st;
  __shared__ uint32_t pick_part[kCompactThreads];
  __shared__ int64_t first_tile;
  __shared__ uint2 stage[kCompactThreads * 16];
  const SegView sv = seg_view(p, blockIdx.y);
  const SelState* __restrict__ stp = sv.st;
  const uint32_t zero_below = zeroed_above(stp);
  if (*p.err) return;
  const bool list_known = ALWAYS_LIST || stp->compact_level == 1u;
  // tiles are handed out by a counter, so blocks beyond the number of list tiles are not needed
  if (list_known && (uint64_t)blockIdx.x * (kCompactThreads * (long_list(stp->list_count, p.k_all) ? 16 : 8)) >=
                        (uint64_t)stp->list_count)
    return;
  // (the first tile's number comes while the digits are replayed)
  if (list_known && threadIdx.x == 0) first_tile = (int64_t)atomicAdd(sv.counters + 2, 1u);
  derive_state<kCompactThreads>(sv, st, 3, pick_part, p.err);
  if (!ALWAYS_LIST && st.compact_level == 3u) {
    compact_body<true>(p, sv, st, 3, 1, zero_below);
    return;
  }
  if (!list_known) {
    if (threadIdx.x == 0) first_tile = (int64_t)atomicAdd(sv.counters + 2, 1u);
    __syncthreads();
  }
  if (long_list(st.list_count, p.k_all))
    list_final_body<16>(p, sv, st, zero_below, first_tile, stage);
  else
    list_final_body<8>(p, sv, st, zero_below, first_tile, stage);
}

// ---------------------------------------------------------------------------
// k_list_hist : histogram of digit `digit` (1 or 2) over the candidates in the
// survivor list; runs only when the list was written at level 1 or from the
// mask.  Digit 1 is needed only for a list written from the mask (k_compact1
// counts it on the way); for digit 2 the digit-1 pick is replayed from hist1 in
// the prologue.
// ---------------------------------------------------------------------------
template <int T>
__device__ __forceinline__ void list_hist_body(const SelParams& p, int digit, uint32_t* __restrict__ lh) {
  constexpr int PER = 8192 / T;  // entries per thread and round
  __shared__ SelState st;
  __shared__ uint32_t pick_part[T];
  const SegView sv = seg_view(p, blockIdx.y);
  if (sv.st->compact_level != 1u || *p.err) return;
  if (digit == 1 && sv.st->use_mask == 0u) return;
  const int tid = threadIdx.x;
  const uint32_t cnt = sv.st->list_count;
  // 8192 entries per block and round; no more blocks than that needs
  uint32_t nb = (cnt + 8191u) / 8192u;
  if (nb > gridDim.x) nb = gridDim.x;
  if (blockIdx.x >= nb) return;
  if (digit == 2) {
    derive_state<T>(sv, st, 2, pick_part, p.err);
  } else {
    if (tid == 0) st = *sv.st;
    __syncthreads();
  }
  const int nbins = (int)digit_mask(digit) + 1;
  for (int b = tid; b < nbins; b += T) lh[b] = 0u;
  __syncthreads();
  const uint32_t klo = st.lo, khi = st.hi;
  const int sh = digit_shift(digit);
  const uint32_t dm = digit_mask(digit);
  for (uint64_t base = (uint64_t)blockIdx.x * 8192u; base < cnt; base += (uint64_t)nb * 8192u) {
    uint32_t key[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {  // (no branch around the loads: behind the list they re-read its last entry)
      const uint64_t q = base + (uint64_t)i * T + tid;
      key[i] = sv.list[q < cnt ? q : cnt - 1u].y & kKeyMask;
    }
#pragma unroll
    for (int i = 0; i < PER; ++i)
      if (base + (uint64_t)i * T + tid < cnt && key[i] >= klo && key[i] <= khi)
        atomicAdd(&lh[(key[i] >> sh) & dm], 1u);
  }
  __syncthreads();
  uint32_t* __restrict__ dst = digit == 1 ? sv.hist1 : sv.hist2;
  for (int b = tid; b < nbins; b += T) {
    const uint32_t v = lh[b];
    if (v) atomicAdd(&dst[b], v);
  }
}

__global__ void __launch_bounds__(256)
k_list_hist(SelParams p, int digit) {
  __shared__ uint32_t lh[kHistBins];
  list_hist_body<256>(p, digit, lh);
}

template <int WAVES, int R>
__global__ void __launch_bounds__(64 * WAVES)
k_compact1(SelParams p) {
  __shared__ uint32_t lh[kHistBins];
  compact1_body<WAVES, R>(p, lh);
}

// ---------------------------------------------------------------------------
// k_level1 : the kernel behind the first pick on the guess route.  If the list was
// written from the mask it counts the second digit over the list's candidates; if the
// guess did not hold it is the level-1 compaction of the histogram route.  8 waves behind the
// marking of vectors that are only read, whose chunks are twice as long: 400 M values of one
// top digit 308 us with 8, 312 with 4, 25.6 M 31 against 44.
// ---------------------------------------------------------------------------
template <int WAVES>
__global__ void __launch_bounds__(64 * WAVES)
k_level1(SelParams p) {
  __shared__ uint32_t lh[kHistBins];
  if (seg_view(p, blockIdx.y).st->use_mask != 0u)
    list_hist_body<64 * WAVES>(p, 1, lh);
  else
    compact1_body<WAVES, kC1R>(p, lh);
}

// ---------------------------------------------------------------------------
// k_level2 : the kernel between the level-1 pass and k_final where the deeper array
// passes exist.  If a list was written at level 1 (or from the mask) it counts the
// last digit over the list's candidates; if the level-1 survivors did not fit one it
// is the level-2 pass over the array (which writes the list if its survivors fit, and
// counts the last digit on the way).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(kCompactThreads)
k_level2(SelParams p) {
  const SegView sv = seg_view(p, blockIdx.y);
  if (*p.err) return;
  if (sv.st->compact_level == 1u) {
    __shared__ uint32_t lh[kHistBins];
    list_hist_body<kCompactThreads>(p, 2, lh);
  } else {
    __shared__ SelState st;
    __shared__ uint32_t pick_part[kCompactThreads];
    derive_state<kCompactThreads>(sv, st, 2, pick_part, p.err);
    compact_body<false>(p, sv, st, 2, 0, kKeyMask);
  }
}


// ---------------------------------------------------------------------------
// Blocks of one launch that wait for each other (k_tail, k_small_step).  The launch's work is cut into units, one for each
// block, and a wait is for all units to be through with a part of it.  Nothing depends on how many blocks run at a time: a
// block takes its unit with its first instructions (meet_take), and one that comes late finds it taken and leaves; before
// the first wait a block that has looked kHelpLooks times takes on units that nobody has, one after the other
// (meet_help), until all are taken.  Every unit then belongs to a block that runs, and those wait for no other.
//   What blocks hand on goes through store_through, load_through and atomics, which are served behind the XCDs' own caches.
// meet_arrive waits until this wave's have been (s_waitcnt vmcnt(0)), then for the block's other waves, and only then counts
// the unit; loads behind meet_wait are issued after it has seen the count.  The orders that the language knows (a release
// in front of the count, an acquire behind the look) would do the same and besides write back and invalidate the whole
// cache once for every wave: 72 us instead of 28 on a step of 1 M x 4.
//   Beside a stream of copies, whose blocks leave no compute unit empty for long, many blocks start late.  List kernels / 256
// looks before every unit and one lane searching for it / 64 before the first and all lanes searching, us: select 25.6 M
// 157/345/130, 138 M 325/607/283, step 11.7 M x 8 559/646/508, 3 M x 2 variance rule 145/264/115 (beside variances of 268 M
// values 282/260/228, 578/343/342, 676/628/624, 198/254/229; beside matrix products 5 to 10 % less than the list kernels).
// 16 looks take on units whose blocks are about to start: 1 M x 4 beside steps of 134 M x 2 100, else 53.
// ---------------------------------------------------------------------------
constexpr int kMeetWords = 8;   // words that the units of a wait are counted on,
constexpr int kMeetLine = 32;   // so many words apart
constexpr int kMeetWait = kMeetWords * kMeetLine;
constexpr int kHelpLooks = 64;

struct Meeting {
  uint32_t* claim;  // [units] `mark`: somebody has taken the unit
  uint32_t* count;  // [waits][kMeetWait] units that are through, zero at first
  uint32_t mark;
  int units;
};

#ifdef ARTOPK_HELD_BLOCKS
// A build for tests: two blocks in three start late, and waits expire after a number of looks that the test sets.
struct HeldBlocks {
  uint32_t ticks;   // of 10 ns
  uint32_t looks;   // instead of kSpinLimit
  uint32_t helped;  // units taken on for others so far
};
__device__ HeldBlocks held_blocks;
__device__ __forceinline__ void meet_start() {
  if ((blockIdx.x + blockIdx.y) % 3u != 0u) {
    const uint64_t from = wall_clock64();
    for (int i = 0; i < (1 << 16) && wall_clock64() - from < held_blocks.ticks; ++i) __builtin_amdgcn_s_sleep(2);
  }
}
__device__ __forceinline__ int meet_limit() { return (int)held_blocks.looks; }
__device__ __forceinline__ void meet_helped() { atomicAdd(&held_blocks.helped, 1u); }
#else
__device__ __forceinline__ void meet_start() {}
__device__ __forceinline__ int meet_limit() { return kSpinLimit; }
__device__ __forceinline__ void meet_helped() {}
#endif

// What comes from on-chip memory and is the same in every lane, taken as such: addresses and loops stay scalar.
template <typename V>
__device__ __forceinline__ V same(V v) {
  return (V)__builtin_amdgcn_readfirstlane((int)v);
}
template <typename V>
__device__ __forceinline__ V* same_ptr(V* q) {
  const uint64_t v = (uint64_t)q;
  return (V*)(((uint64_t)same((uint32_t)(v >> 32)) << 32) | same((uint32_t)v));
}

// Whether unit u was still to be had; one lane calls it.
__device__ __forceinline__ bool meet_take(const Meeting& m, int u) {
  return __hip_atomic_exchange(&m.claim[u], m.mark, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != m.mark;
}

// Unit u is through with the part in front of wait b; all threads of the block call it.
__device__ __forceinline__ void meet_arrive(const Meeting& m, int b, int u) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0)
    __hip_atomic_fetch_add(&m.count[b * kMeetWait + u % kMeetWords * kMeetLine], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Waits for `total` units, at most for 1 + looks looks; whether they are there.  If they are not in the end (meet_limit, a
// second or so), the block sets the error word and leaves: blocks that come later leave at once, those that wait for its
// units or theirs when their looks are used up, and artopk_status reports it and clears what the launch leaves behind.  All
// threads of the block call it; sh is a word of on-chip memory, free before and after.
__device__ __forceinline__ bool meet_wait(const Meeting& m, int b, int total, int looks, int& sh) {
  if (same(threadIdx.x >> 6) == 0u) {
    const uint32_t lane = lane_id();
    bool ok = false;
    for (int i = 0; !ok && i <= looks; ++i) {
      uint32_t v = lane < (uint32_t)kMeetWords ? load_through(&m.count[b * kMeetWait + lane * kMeetLine]) : 0u;
      v += __shfl_xor(v, 1, 64);
      v += __shfl_xor(v, 2, 64);
      v += __shfl_xor(v, 4, 64);
      ok = same(v) == (uint32_t)total;
    }
    if (lane == 0u) sh = ok ? 1 : 0;
  }
  __syncthreads();
  const bool ok = same(sh) != 0;
  __syncthreads();
  return ok;
}

// A unit that nobody had taken and that this block has now, searched for from `look` on, or -1.  helped (or nullptr) counts
// them, before each is taken: a late block that finds its own taken finds it counted.  All threads of the block call it.
__device__ __forceinline__ int meet_help(const Meeting& m, int look, uint32_t* helped, int& sh) {
  if (same(threadIdx.x >> 6) == 0u) {
    const int lane = (int)lane_id();
    int got = -1;
    for (int i = 0; i < m.units && got < 0; i += 64) {
      const int u = (look + i + lane) % m.units;
      uint64_t open = __ballot(i + lane < m.units && load_through(&m.claim[u]) != m.mark);
      for (; open != 0ull && got < 0; open &= open - 1ull) {
        const int c = (look + i + __builtin_ctzll(open)) % m.units;
        int ok = 0;
        if (lane == 0) {
          if (helped) {
            __hip_atomic_fetch_add(helped, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
          }
          ok = meet_take(m, c) ? 1 : 0;
          if (ok)
            meet_helped();
          else if (helped)
            __hip_atomic_fetch_sub(helped, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (same(ok) != 0) got = c;
      }
    }
    if (lane == 0) sh = got;
  }
  __syncthreads();
  const int got = same(sh);
  __syncthreads();
  return got;
}

// ---------------------------------------------------------------------------
// k_tail : a flat selection from the top digits on (or several at a time, one per blockIdx.y), in one launch instead of
// four behind a pass that counted the top digits (pick, compaction, list digits, final pass), six behind the read-only
// marking or five behind nothing.  Those are bound by latency, 5 us for a launch and a trip to memory or two in each; here
// the blocks wait for each other in between (a microsecond), and a block's survivors (keys that reach the threshold's
// top digit, or the guessed bound) stay on chip, an eighth with each wave, in order.  List kernels / this, us: select 138 M,
// one in a hundred kept 181 / 170 (now 160), with values in runs 402 / 174, all equal 1914 / 1209; 8 selections on 25.6 M
// 278 / 248 (now 219 with their norms);
// variance rule, pass and selection, 11.7 M x 8 312 / 281, all equal 658 / 576.
//   kTailSpans: the pieces of k_mark_spans, if their bound holds (k_pick_mask's rule).  How many there are in front of
// every chunk is known, so each wave has as many as any other, however they are spread.  kTailHist: the top digits' counts
// of a fused pass; kTailNone (and a bound that does not hold): nothing, the blocks count them first.  Each wave then has as
// many elements as any other, in up to 16 pieces (64 where several vectors share the blocks) spread over the vector, so
// that large values that lie together are those of many waves.  In one piece, a few waves had most of the work (variance
// rule, 11.7 M x 2, one in a hundred, list kernels / one piece / now: normal values 131/122/124, layers of 54 scales
// 132/133/124, a run 163/195/152, sorted 222/251/203; x 8 312/284/281, 298/281/271, 311/331/286, 528/532/478).
//   What a wave does not keep on chip goes to its part of the list's memory (of the pieces it always fits; with a limit of
// 2000 entries a wave instead, 60 M x 4 and one in a hundred kept had read the vectors again: 642 us, by the list kernels
// 318, now 287); survivors that do not fit there either are read from the vector again each time.
//   The blocks count the threshold's next digit over their survivors, wait, pick it each for itself, and so on.  Where no
// more than 512 candidates are left for the last digit (without many ties: 13 of 11.7 M normal values), each block hands
// on its own, and how many entries lie above them in each of its pieces; else it counts their digits, waits, and counts
// then what is kept.  Either way every wave knows what is kept in front of each of its pieces and writes its own.  A block
// that has waited for the first counts for a while takes on ranges that nobody has and collects them anew each time (see
// k_small_step: nothing depends on how many blocks run at a time).
//   The length of the code matters: it is read in by a launch of 40 us.  With rows and entries taken by instructions of
// their own eight and four at a time, 108 KB, the same took 15 us longer behind a pass than in 29 KB.
// row_log2: rows of 256 elements in a piece.  grid = (ranges, vectors), block = 64 kTailWaves.  The counts lie in the
// segment's scratch block (cleared before), what the blocks hand on in S's memory.
// ---------------------------------------------------------------------------
constexpr int kTailSpans = 0, kTailHist = 1, kTailNone = 2;
constexpr int kTailRanges = 256;   // blocks of a launch, at most: one per compute unit
constexpr int kTailWaves = 8;      // (16 a block: 87 registers of each thread spilled, and everything took 35 us longer)
constexpr int kTailKeep = 2000;    // survivors a wave keeps on chip
constexpr int kTailRow = 256;
constexpr int kTailPieces = 64;  // pieces of a wave's elements, at most
constexpr int kTailFew = 64 * kTailWaves;  // candidates that are handed on one by one, a few of each range in places of its own
constexpr int kTailSlots = 4;
constexpr int kTailWaits = 4;
// in the words of kSegHist2 behind the last digit's 128 counts: whether somebody has taken a range, the waits' counters
constexpr int kTailClaim = 128, kTailCount = 512;
constexpr int kTailFewAt = kTailWaits * kMeetWait;  // (behind kTailCount: candidates handed on so far)
static_assert(kTailClaim + kTailRanges <= kTailCount && kTailCount + kTailFewAt < kHistBins, "they fit");

// Adds 1 to hist[bin] for every active lane; lanes with the first one's bin (all, where values are equal) in one addition.
__device__ __forceinline__ void wave_count(uint32_t* hist, uint32_t bin) {
  const uint32_t one = __builtin_amdgcn_readfirstlane(bin);
  const uint64_t same = __ballot(bin == one);
  if (bin != one)
    atomicAdd(&hist[bin], 1u);
  else if (popc_lt(same) == 0u)
    atomicAdd(&hist[one], (uint32_t)__popcll(same));
}

// A wave's walk over rows of 256 elements of x, four a lane, eight of them in flight: at(r) is the first element of row r,
// a multiple of 4, n or more where there is no such row.  row(its number, the lane's first element, words) for every row in
// order, with what lies behind n unspecified, until enough() is true after eight of them.  OWN: each of the eight is taken
// by instructions of its own, which pays for vectors of many rows (all equal, 138 M: 1209 us, else 1309); else by the same
// ones.  x16: 16 bytes to read where n has not even those.  The 64 lanes of a wave call it.
typedef uint32_t RowWords __attribute__((ext_vector_type(32)));

template <bool OWN, typename At, typename Row, typename Enough>
__device__ __forceinline__ void wave_walk(const float* __restrict__ x, uint32_t n, const void* x16, int nrows, At at,
                                          Row row, Enough enough) {
  const uint32_t lane = lane_id();
  const uint32_t last = n & ~3u;  // the group that n cuts, if it does
  uint4 cut = make_uint4(0u, 0u, 0u, 0u);
  if (last + 0 < n) cut.x = __float_as_uint(x[last + 0]);
  if (last + 1 < n) cut.y = __float_as_uint(x[last + 1]);
  if (last + 2 < n) cut.z = __float_as_uint(x[last + 2]);
  const float* const from = n >= 4u ? x : static_cast<const float*>(x16);
  const uint32_t most = n >= 4u ? last - 4u : 0u;
  for (int r0 = 0; r0 < nrows && !enough(); r0 += 8) {
    uint4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const uint32_t j = at(r0 + u) + 4u * lane;
      v[u] = *reinterpret_cast<const uint4*>(from + (j < most ? j : most));
    }
    if (OWN) {
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const uint32_t j = at(r0 + u) + 4u * lane;
        if (j == last) v[u] = cut;
        if (r0 + u < nrows) row(r0 + u, j, v[u]);
      }
      continue;
    }
    RowWords w;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      w[4 * u + 0] = v[u].x;
      w[4 * u + 1] = v[u].y;
      w[4 * u + 2] = v[u].z;
      w[4 * u + 3] = v[u].w;
    }
#pragma unroll 1
    for (int u = 0; u < 8 && r0 + u < nrows; ++u) {
      const uint32_t j = at(r0 + u) + 4u * lane;
      uint4 t = make_uint4(w[4 * u], w[4 * u + 1], w[4 * u + 2], w[4 * u + 3]);
      if (j == last) t = cut;
      row(r0 + u, j, t);
    }
  }
}

// The elements of a wave's rows (see wave_walk) whose key reaches `bound`, in order, the first cap of them: put(number,
// element, raw bits); returns their number, or more than cap.
template <bool OWN, typename At, typename Put>
__device__ __forceinline__ uint32_t wave_collect(const float* __restrict__ x, uint32_t n, const void* x16, int nrows, At at,
                                                 uint32_t bound, SpanQueue& qu, uint32_t cap, Put put) {
  const uint32_t lane = lane_id();
  uint32_t count = 0u, head = 0u, queued = 0u;
  auto take = [&](uint32_t m) __attribute__((always_inline)) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const uint32_t p = (head + lane) & 127u;
    const uint4 v = qu.val[p];
    const uint32_t g = qu.group[p];
    const uint32_t raw[4] = {v.x, v.y, v.z, v.w};
    uint32_t own = 0u;
#pragma unroll
    for (int e = 0; e < 4; ++e) own |= (raw[e] & kKeyMask) >= bound && 4u * g + e < n ? 1u << e : 0u;
    if (lane >= m) own = 0u;
    const uint32_t c = (uint32_t)__popc(own);
    uint32_t before = 0u, total = 0u;
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      const uint64_t plane = __ballot((c >> b) & 1u);
      before += popc_lt(plane) << b;
      total += (uint32_t)__popcll(plane) << b;
    }
    uint32_t pos = count + before;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if ((own >> e) & 1u) {
        if (pos < cap) put(pos, 4u * g + e, raw[e]);
        ++pos;
      }
    }
    count += total;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  wave_walk<OWN>(x, n, x16, nrows, at, [&](int, uint32_t j, uint4 raw) __attribute__((always_inline)) {
    // (take() looks which of a group's elements there are)
    const uint32_t a = raw.x & kKeyMask, b = raw.y & kKeyMask, c = raw.z & kKeyMask, d = raw.w & kKeyMask;
    const uint32_t ab = a > b ? a : b, cd = c > d ? c : d;
    const bool hit = (ab > cd ? ab : cd) >= bound && j < n;
    const uint64_t hits = __ballot(hit);
    if (hits == 0ull) return;
    if (hit) {
      const uint32_t p = (head + queued + popc_lt(hits)) & 127u;
      qu.val[p] = raw;
      qu.group[p] = j >> 2;
    }
    queued += (uint32_t)__popcll(hits);
    if (queued >= 64u) {
      take(64u);
      head += 64u;
      queued -= 64u;
    }
  }, [&]() __attribute__((always_inline)) { return count > cap; });  // (no use in going on)
  if (queued != 0u) take(queued);
  return count;
}

struct TailShared {
  uint2 list[kTailWaves][kTailKeep];  // (element, raw bits)
  union {
    __attribute__((aligned(16))) uint32_t hist[kHistBins];
    SpanQueue qu[kTailWaves];
    struct {  // kept entries: (above the threshold, at it)
      uint2 own[kTailWaves][kTailPieces];    // of a wave's piece
      uint2 front[kTailWaves][kTailPieces];  // in front of it, less those of the wave's pieces before
      uint64_t all[kTailPieces];             // of all blocks' pieces of that number: above << 32 | at
      uint64_t before[kTailPieces];          // of those, the blocks in front of this one's
      uint2 few[kTailFew];                   // candidates: (place, last digit)
    } kept;
  } pool;
  uint32_t tail[128];
  SelState st, st1;
  uint32_t part[kTailWaves];
  uint16_t owned[kTailRanges];
  int verdict;
  uint32_t few_n, few_at;
  uint2 few_all[kTailFew];         // all blocks' candidates, where there are few
  uint32_t chunk_at[kMaxChunks + 1];  // entries in front of every chunk of the marking (kTailSpans)
};

// k_tail's work.  full: behind a marking whose bound does not hold.  bound, total: kTailSpans' bound and the number of
// entries that reach it.
template <int source, bool full>
__device__ __forceinline__ void tail_select(const SelParams& p, const SegView& sv, TailShared& sh, int row_log2,
                                            uint32_t bound, uint32_t total) {
  constexpr int WAVES = kTailWaves, T = 64 * WAVES, BPT = kHistBins / T;
  constexpr bool spans = source == kTailSpans;
  auto& list = sh.list;
  auto& pool = sh.pool;
  auto& tail = sh.tail;
  auto& st = sh.st;
  auto& st1 = sh.st1;
  auto& part = sh.part;
  auto& owned = sh.owned;
  auto& verdict = sh.verdict;
  auto& few_n = sh.few_n;
  auto& few_at = sh.few_at;
  auto& few_all = sh.few_all;
  auto& chunk_at = sh.chunk_at;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nranges = gridDim.x, vec = blockIdx.y, c0 = blockIdx.x;
  const float* x = sv.x;
  const uint32_t n = (uint32_t)p.n;
  const uint32_t k = sv.d.k;
  uint32_t* const count = sv.hist2 + kTailCount;
  const Meeting meet{sv.hist2 + kTailClaim, count, 1u, nranges};
  // the wave's pieces of range c: `pieces` of them, 256 << row_log2 elements each, `stride` elements apart
  const uint32_t stride = ((uint32_t)nranges * WAVES) << (8 + row_log2);
  const int pieces = (int)((n + stride - 1u) / stride), nrows = pieces << row_log2;
  auto rows_of = [&](int c) __attribute__((always_inline)) {
    const uint32_t first = (uint32_t)(c * WAVES + wave) << (8 + row_log2);
    return [=](int r) __attribute__((always_inline)) {
      return (uint32_t)(r >> row_log2) * stride + first + ((uint32_t)(r & ((1 << row_log2) - 1)) << 8);
    };
  };
  // kept entries of every range's pieces: [piece][range], above << 32 | at
  uint64_t* const kept_of = reinterpret_cast<uint64_t*>(p.S) + (size_t)vec * kTailPieces * nranges;
  // candidates of every range where there are few: kTailSlots each, and what is more of any: last digit << 32 | place, which
  // is (piece x ranges + range) x waves + wave
  uint64_t* const slots_of = reinterpret_cast<uint64_t*>(p.S) + (size_t)kTailPieces * kTailRanges +
                             (size_t)vec * (kTailRanges * kTailSlots + kTailFew);
  uint64_t* const few_of = slots_of + kTailRanges * kTailSlots;
  if (tid == 0) {
    verdict = meet_take(meet, c0) ? 0 : 1;
    owned[0] = (uint16_t)c0;
    st = SelState{};
    st.hi = kKeyMask;
    st.need = k;
  }
  if (tid < 128) tail[tid] = 0u;
  __syncthreads();
  if (verdict != 0) return;
  int n_owned = 1;

  bool listed = false;
  uint32_t mine = 0u;  // the wave's entries in `list`
  const uint32_t share = spans ? (total + (uint32_t)(nranges * WAVES) - 1u) / (uint32_t)(nranges * WAVES) : 0u;
  // what a wave does not keep on chip goes to its part of the survivor list's memory
  const uint32_t room = sv.d.cap / (uint32_t)(nranges * WAVES);
  // (a share of the pieces' entries, of which there are no more than the list takes, always fits)
  auto more_of = [&](int c) __attribute__((always_inline)) { return sv.list + (size_t)(c * WAVES + wave) * room; };
  auto put = [&](int c, uint32_t m, uint2 v) __attribute__((always_inline)) {
    if (m < (uint32_t)kTailKeep)
      list[wave][m] = v;
    else
      more_of(c)[m - kTailKeep] = v;
  };
  int cur = -1;  // the range whose survivors `list` holds, if they fit
  // The survivors of range c, from the pieces or from the vector; all threads call it.
  auto collect = [&](int c) __attribute__((always_inline)) {
    cur = c;
    mine = 0u;
    __syncthreads();  // (`pool` is free)
    // entries [e0, e1) of all, in order: this wave's (from the vector: what it has room for)
    const uint64_t from = (uint64_t)((uint32_t)c * WAVES + (uint32_t)wave) * share;
    const uint32_t e0 = from < total ? (uint32_t)from : total;
    const uint32_t e1 = !spans ? (uint32_t)kTailKeep + room : total - e0 < share ? total : e0 + share;
    int ch = 0;  // the chunk of entry e0: the last with no more entries in front of it
    if (spans) {
#pragma unroll
      for (int w = kMaxChunks / 2; w > 0; w >>= 1) ch += same(chunk_at[ch + w]) <= e0 ? w : 0;
    }
    const uint32_t span = (uint32_t)p.tiles.span, nspans = spans ? (n + span - 1u) / span : 1u;
    uint32_t at = spans ? same(chunk_at[ch]) : 0u;  // entries in front of span s0
    for (uint32_t s0 = spans ? (uint32_t)ch * same((uint32_t)sv.d.geom.chunk_elems) / span : 0u; s0 < nspans && at < e1; s0 += 64u) {
      uint32_t cnt = 0u, incl = 0u;
      uint64_t read = 1ull;  // what has to be taken from the vector: the wave's rows, or spans with more than their pieces hold
      if (spans) {
        cnt = s0 + (uint32_t)lane < nspans ? sv.tcnt[s0 + (uint32_t)lane] : 0u;
        incl = wave_incl_scan(cnt);
        const uint64_t some = __ballot(at + incl > e0 && at + incl - cnt < e1 && cnt != 0u);
        read = some & __ballot(cnt > (uint32_t)sv.tcap);
        // eight rows of 64 entries in flight, whosever piece they are of (the first 64 of four pieces at a time, and each
        // further row of theirs behind the one before: 8 selections of 25.6 M, 123 entries a piece, 10.5 us here, now 7.8)
        uint64_t left = some & ~read;
        const uint2* piece = sv.tbuf;
        uint32_t first = 0u, m0 = 0u, m1 = 0u;  // of the piece: the number of its first entry; its entries [m0, m1) are to come
        while (left != 0ull || m0 < m1) {
          uint2 ent[8];
          uint32_t number[8], there[8];
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            if (m0 >= m1 && left != 0ull) {
              const int s = __builtin_ctzll(left);
              left &= left - 1ull;
              m1 = (uint32_t)__builtin_amdgcn_readlane((int)cnt, s);
              first = at + (uint32_t)__builtin_amdgcn_readlane((int)(incl - cnt), s);
              piece = sv.tbuf + (size_t)(s0 + (uint32_t)s) * (size_t)sv.tcap;
              m0 = e0 > first ? e0 - first : 0u;
              if (m1 > e1 - first) m1 = e1 - first;
            }
            number[q] = first + m0 - e0;
            there[q] = m0 < m1 ? m1 - m0 : 0u;
            ent[q] = piece[(uint32_t)lane < there[q] ? m0 + (uint32_t)lane : 0u];
            m0 += 64u;
          }
#pragma unroll
          for (int q = 0; q < 8; ++q)
            if ((uint32_t)lane < there[q]) put(c, number[q] + (uint32_t)lane, ent[q]);
        }
      }
      for (; read != 0ull; read &= read - 1ull) {
        const int s = __builtin_ctzll(read);
        const uint32_t first = at + (uint32_t)__builtin_amdgcn_readlane((int)(incl - cnt), s);
        const uint32_t x0 = (s0 + (uint32_t)s) * span, x1 = spans && n - x0 > span ? x0 + span : n;
        const auto own = rows_of(c);
        const uint32_t found = wave_collect<spans || full>(
            x, x1, p.zero_base, spans ? (int)((x1 - x0 + 255u) / 256u) : nrows,
            [&](int r) __attribute__((always_inline)) { return spans ? x0 + 256u * (uint32_t)r : own(r); },
            bound, pool.qu[wave], spans ? e1 - first : e1, [&](uint32_t m, uint32_t j, uint32_t raw) __attribute__((always_inline)) {
              const uint32_t e = first + m;
              if (e >= e0 && e < e1) put(c, e - e0, make_uint2(j, raw));
            });
        if (!spans) mine = found;
      }
      at += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    }
    if (spans) mine = e0 < e1 ? e1 - e0 : 0u;
    __syncthreads();
    mine = same(mine);
    listed = mine <= (uint32_t)kTailKeep + room;
  };
  auto entry = [&](int c, uint32_t i) __attribute__((always_inline)) {
    return i < (uint32_t)kTailKeep ? list[wave][i] : more_of(c)[i - kTailKeep];
  };
  // use(element, raw bits) for every survivor of range c, and others below the bound, in some thread
  auto each = [&](int c, auto use) __attribute__((always_inline)) {
    if (spans || (listed && c == cur)) {
      for (uint32_t q0 = 0u; q0 < mine; q0 += 256u) {  // four entries in flight
        uint2 ent[4];
#pragma unroll
        for (uint32_t q = 0u; q < 4u; ++q) {
          const uint32_t i = q0 + 64u * q + (uint32_t)lane;
          ent[q] = entry(c, i < mine ? i : mine - 1u);
        }
        if (spans) {
#pragma unroll
          for (uint32_t q = 0u; q < 4u; ++q)
            if (q0 + 64u * q + (uint32_t)lane < mine) use(ent[q].x, ent[q].y);
          continue;
        }
#pragma unroll 1
        for (uint32_t m = q0; m < mine && m < q0 + 256u; m += 64u) {
          if (m + (uint32_t)lane < mine) use(ent[0].x, ent[0].y);
#pragma unroll
          for (int q = 0; q < 3; ++q) ent[q] = ent[q + 1];
        }
      }
    } else {
      wave_walk<full>(x, n, p.zero_base, nrows, rows_of(c), [&](int, uint32_t j, uint4 v) __attribute__((always_inline)) {
        const uint32_t raw[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (uint32_t e = 0u; e < 4u; ++e)
          if (j + e < n) use(j + e, raw[e]);
      }, []() { return false; });
    }
  };
  auto report_state = [&]() __attribute__((always_inline)) {  // what select_info reports: the state behind the top digit
    st1 = st;
    st1.compact_level = spans || fits_list(st, sv.d.cap) ? 1u : 0u;
    st1.list_count = spans ? total : st1.compact_level ? st.n_gt + st.cand : 0u;
    st1.use_mask = spans ? 1u : 0u;
    st1.list_lo = spans ? bound : 0u;
    st1.need_full = full ? 1u : 0u;
  };
  // the piece that element j of a wave's belongs to (exact: fewer than 2^20 steps of 2048 << row_log2 elements)
  const float per_piece = 1.0f / (float)nranges;
  auto piece_of = [&](uint32_t j) __attribute__((always_inline)) {
    static_assert(WAVES == 8, "a block's pieces of one number: 2048 << row_log2 elements");
    return spans ? 0u : (uint32_t)(((float)(j >> (11 + row_log2)) + 0.5f) * per_piece);
  };
  const int kept_pieces = spans ? 1 : pieces;
  auto give_up = [&]() __attribute__((always_inline)) {
    if (tid == 0) atomicOr(p.err, kErrWait);
    __builtin_amdgcn_wave_barrier();  // (the lanes meet here, not where the ways out of the loops do: those stay scalar)
  };

  constexpr bool counted = source == kTailHist;  // the top digits' counts are there
  bool few = false;
  uint32_t cand = 0u;      // candidates of the last digit
  uint64_t ahead[kTailRanges / 64];  // kept_of of the wave's first piece, on its way while the threshold is picked
  // 0: the top digits of the survivors, or of everything where no bound is known yet; 1: the second digits of the
  // candidates; 2: the last ones; 3: how many are kept of every piece; 4: the outputs
  for (int stage = 0;; ++stage) {
    const uint32_t klo = same(st.lo), khi = same(st.hi), quota = same(st.need);
    uint32_t* const dst = stage == 0 ? sv.hseg : stage == 1 ? sv.hist1 : sv.hist2;
    const bool digits = stage < 2 || (stage == 2 && !few);
    const int sh_bits = digit_shift(stage), bins = (int)digit_mask(stage) + 1;
    for (int done = 0, look = c0 + 1; stage > 0 || !counted;) {
      for (; done < n_owned; ++done) {
        const int c = same((int)owned[done]);
        if (c != cur && (spans || stage > 0)) collect(c);
        const bool again = stage == 4 && n_owned > 1;  // (the last range's counts are there else)
        if (stage < 4 || again) {
          // the digits of the candidates, or the entries of the wave's pieces that reach klo (with a few candidates at
          // stage 2 also these themselves)
          __syncthreads();
          if (digits) {
            for (int i = tid; i < kHistBins / 4; i += T) reinterpret_cast<uint4*>(pool.hist)[i] = make_uint4(0u, 0u, 0u, 0u);
          } else {
            if (lane < kept_pieces) pool.kept.own[wave][lane] = make_uint2(0u, 0u);
            if (tid == 0) few_n = 0u;
          }
          __syncthreads();
          auto digit = [&](uint32_t kk) __attribute__((always_inline)) {
            if (kk >= klo && kk <= khi) wave_count(pool.hist, (kk >> sh_bits) & (uint32_t)(bins - 1));
          };
          auto hand_on = [&](uint32_t q, uint32_t kk) __attribute__((always_inline)) {
            const uint32_t i = atomicAdd(&few_n, 1u);
            if (i < (uint32_t)kTailFew)
              pool.kept.few[i] = make_uint2((q * (uint32_t)nranges + (uint32_t)c) * WAVES + (uint32_t)wave, kk & 0x7fu);
          };
          uint32_t upA = 0u, atB = 0u;
          if (spans && digits) {
            each(c, [&](uint32_t, uint32_t raw) __attribute__((always_inline)) { digit(raw & kKeyMask); });
          } else if (spans) {
            each(c, [&](uint32_t, uint32_t raw) __attribute__((always_inline)) {
              const uint32_t kk = raw & kKeyMask;
              if (kk > khi) {
                ++upA;
              } else if (kk >= klo) {
                ++atB;
                if (stage == 2) hand_on(0u, kk);
              }
            });
          } else {
            each(c, [&](uint32_t j, uint32_t raw) __attribute__((always_inline)) {
              const uint32_t kk = raw & kKeyMask;
              if (digits) return digit(kk);
              if (kk < klo) return;
              const uint32_t q = piece_of(j);
              if (stage == 2 && kk <= khi) hand_on(q, kk);
              for (bool left = true; left;) {  // (in order: the 64 lanes hold one piece's, or a few pieces')
                const uint32_t one = __builtin_amdgcn_readfirstlane(q);
                const uint64_t with = __ballot(q == one), up = __ballot(q == one && kk > khi);
                if (q == one) {
                  if (popc_lt(with) == 0u) {
                    const uint32_t a = (uint32_t)__popcll(up);
                    atomicAdd(&pool.kept.own[wave][one].x, a);
                    atomicAdd(&pool.kept.own[wave][one].y, (uint32_t)__popcll(with) - a);
                  }
                  left = false;
                }
              }
            });
          }
          if (spans && !digits) {
            const uint64_t both = wave_allsum_u64(((uint64_t)upA << 32) | atB);
            if (lane == 0) pool.kept.own[wave][0] = make_uint2((uint32_t)(both >> 32), (uint32_t)both);
          }
          __syncthreads();
        }
        if (digits) {
          for (int i = tid; i < bins; i += T) {
            const uint32_t v = pool.hist[i];
            if (v) atomicAdd(&dst[i], v);
          }
          meet_arrive(meet, stage, c);
          continue;
        }
        if (stage == 2) {
          const uint32_t mine_few = same(few_n < (uint32_t)kTailFew ? few_n : (uint32_t)kTailFew);
          if (tid < kTailSlots) {
            const uint2 f = pool.kept.few[tid];
            store_through(&slots_of[c * kTailSlots + tid], (uint32_t)tid < mine_few ? ((uint64_t)f.y << 32) | f.x : ~(uint64_t)0);
          }
          if (mine_few > (uint32_t)kTailSlots) {
            const uint32_t more = mine_few - (uint32_t)kTailSlots;
            if (tid == 0)
              few_at = __hip_atomic_fetch_add(&count[kTailFewAt], more, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            if ((uint32_t)tid < more && few_at + (uint32_t)tid < (uint32_t)kTailFew) {
              const uint2 f = pool.kept.few[kTailSlots + tid];
              store_through(&few_of[few_at + (uint32_t)tid], ((uint64_t)f.y << 32) | f.x);
            }
          }
        }
        if (stage < 4) {
          if (tid < kept_pieces) {
            uint64_t sum = 0ull;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) sum += ((uint64_t)pool.kept.own[w][tid].x << 32) | pool.kept.own[w][tid].y;
            store_through(&kept_of[(size_t)tid * nranges + c], sum);
          }
          meet_arrive(meet, stage, c);
          continue;
        }
        // kept in front of every piece of the wave's
        for (int q = wave, turn = 0; q < kept_pieces; q += WAVES, ++turn) {
          uint64_t all = 0ull, before = 0ull;
#pragma unroll
          for (int i = 0; i < kTailRanges / 64; ++i) {
            const int r = lane + 64 * i;
            uint64_t v = 0ull;
            if (turn == 0)
              v = ahead[i];
            else if (r < nranges)
              v = load_through(&kept_of[(size_t)q * nranges + r]);
            if (few) v &= ~0xffffffffull;
            all += v;
            before += r < c ? v : 0ull;
          }
          all = wave_allsum_u64(all);
          before = wave_allsum_u64(before);
          if (lane == 0) {
            pool.kept.all[q] = all;
            pool.kept.before[q] = before;
          }
        }
        __syncthreads();
        if (few) {  // (candidates above the threshold, or at it)
          if (!again) {
            if (lane < kept_pieces) pool.kept.own[wave][lane].y = 0u;
            __syncthreads();
          }
          const uint2 f = few_all[tid];
          if ((uint32_t)tid < cand && f.y >= (klo & 0x7fu)) {
            const uint32_t at = f.x / WAVES, q = (at / (uint32_t)nranges) & (uint32_t)(kTailPieces - 1);
            const uint32_t range = at - q * (uint32_t)nranges;
            const bool up = f.y > (klo & 0x7fu);
            const uint64_t v = up ? 1ull << 32 : 1ull;
            atomicAdd(reinterpret_cast<unsigned long long*>(&pool.kept.all[q]), v);
            if (range < (uint32_t)c) atomicAdd(reinterpret_cast<unsigned long long*>(&pool.kept.before[q]), v);
            if (range == (uint32_t)c && !again) {
              uint2* const own = &pool.kept.own[f.x % WAVES][q];
              atomicAdd(up ? &own->x : &own->y, 1u);
            }
          }
          __syncthreads();
        }
        {
          const bool real = lane < kept_pieces;
          uint64_t mine_q = 0ull, front = real ? pool.kept.before[lane] : 0ull;
#pragma unroll
          for (int w = 0; w < WAVES; ++w) {
            const uint2 o = real ? pool.kept.own[w][lane] : make_uint2(0u, 0u);
            const uint64_t v = ((uint64_t)o.x << 32) | o.y;
            front += w < wave ? v : 0ull;
            mine_q = w == wave ? v : mine_q;
          }
          uint64_t all = real ? pool.kept.all[lane] : 0ull, own = mine_q;
          const uint64_t all0 = all;
          all = wave_incl_scan(all);
          own = wave_incl_scan(own);
          front += all - all0;
          own -= mine_q;
          if (real)
            pool.kept.front[wave][lane] =
                make_uint2((uint32_t)(front >> 32) - (uint32_t)(own >> 32), (uint32_t)front - (uint32_t)own);
        }
        __syncthreads();
        uint32_t runA = 0u, runB = 0u;
        auto keep = [&](uint32_t a, uint32_t b, uint32_t j, uint32_t raw) __attribute__((always_inline)) {
          const uint32_t m = a + (b < quota ? b : quota);
          if (m >= k) return;
          sv.idx_out[m] = (int32_t)j;
          if (sv.vals_row) sv.vals_row[m] = __uint_as_float(raw);
        };
        if (spans || listed) {
          for (uint32_t q0 = 0u; q0 < mine; q0 += 256u) {
            uint2 four[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const uint32_t q = q0 + 64u * u + (uint32_t)lane;
              four[u] = entry(c, q < mine ? q : mine - 1u);
            }
#pragma unroll 1
            for (uint32_t m = q0; m < mine && m < q0 + 256u; m += 64u) {
              const bool ok = m + (uint32_t)lane < mine;
              const uint2 ent = four[0];
#pragma unroll
              for (int u = 0; u < 3; ++u) four[u] = four[u + 1];
              const uint32_t kk = ent.y & kKeyMask;
              const bool is_a = ok && kk > khi, is_b = ok && kk >= klo && kk <= khi;
              const uint64_t ma = __ballot(is_a), mb = __ballot(is_b);
              if (is_a || is_b) {
                const uint2 front = pool.kept.front[wave][piece_of(ent.x)];
                const uint32_t a = front.x + runA + popc_lt(ma), b = front.y + runB + popc_lt(mb);
                if (is_a || b < quota) keep(a, b, ent.x, ent.y);
              }
              runA += (uint32_t)__popcll(ma);
              runB += (uint32_t)__popcll(mb);
            }
          }
        } else {
          wave_walk<full>(x, n, p.zero_base, nrows, rows_of(c), [&](int r, uint32_t j, uint4 v) __attribute__((always_inline)) {
              const uint32_t raw[4] = {v.x, v.y, v.z, v.w};
              uint32_t isA = 0u, isB = 0u;
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const uint32_t kk = raw[e] & kKeyMask;
                isA |= j + e < n && kk > khi ? 1u << e : 0u;
                isB |= j + e < n && kk >= klo && kk <= khi ? 1u << e : 0u;
              }
              if (__ballot((isA | isB) != 0u) == 0ull) return;
              const uint32_t cA = (uint32_t)__popc(isA), cB = (uint32_t)__popc(isB);
              const uint2 front = pool.kept.front[wave][r >> row_log2];
              uint32_t a = front.x + runA, b = front.y + runB;
#pragma unroll
              for (int q = 0; q < 3; ++q) {
                const uint64_t pa = __ballot((cA >> q) & 1u), pb = __ballot((cB >> q) & 1u);
                a += popc_lt(pa) << q;
                b += popc_lt(pb) << q;
                runA += (uint32_t)__popcll(pa) << q;
                runB += (uint32_t)__popcll(pb) << q;
              }
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                const bool is_a = (isA >> e) & 1u, is_b = (isB >> e) & 1u;
                if (is_a || (is_b && b < quota)) keep(a, b, j + e, raw[e]);
                a += is_a ? 1u : 0u;
                b += is_b ? 1u : 0u;
              }
          }, []() { return false; });
        }
      }
      if (stage == 4) return;
      const bool first = stage == (counted ? 1 : 0);
      if (meet_wait(meet, stage, nranges, first && look >= 0 ? (n_owned == 1 ? kHelpLooks : 0) : meet_limit(), verdict)) break;
      if (!first || look < 0) return give_up();
      look = meet_help(meet, look, nullptr, verdict);  // (-1: all are taken)
      if (look < 0) continue;
      if (tid == 0) owned[n_owned] = (uint16_t)look;
      __syncthreads();
      ++n_owned;
      ++look;
    }
    if (!digits) {
#pragma unroll
      for (int i = 0; i < kTailRanges / 64; ++i)
        ahead[i] = wave < kept_pieces && lane + 64 * i < nranges
                       ? load_through(&kept_of[(size_t)wave * nranges + lane + 64 * i]) : 0ull;
    }
    if (stage == 3) continue;
    if (stage == 1 && tid == 0) report_state();
    uint32_t h[BPT];
    if (stage == 0 && counted) {
#pragma unroll
      for (int j = 0; j < BPT; ++j) h[j] = 0u;
      for (int r0 = 0; r0 < sv.htop_reps; r0 += 8) {
        uint4 q[8][BPT / 4];
#pragma unroll
        for (int r = 0; r < 8; ++r)
#pragma unroll
          for (int j = 0; j < BPT / 4; ++j)
            q[r][j] = reinterpret_cast<const uint4*>(sv.htop + (size_t)(r0 + r < sv.htop_reps ? r0 + r : r0) * kHistBins)
                [BPT / 4 * tid + j];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          if (r0 + r < sv.htop_reps) {
#pragma unroll
            for (int j = 0; j < BPT / 4; ++j) {
              h[4 * j + 0] += q[r][j].x;
              h[4 * j + 1] += q[r][j].y;
              h[4 * j + 2] += q[r][j].z;
              h[4 * j + 3] += q[r][j].w;
            }
          }
        }
      }
    } else if (stage == 2 && few) {
      constexpr int PER = kTailRanges * kTailSlots / T;
      uint64_t f[PER];
#pragma unroll
      for (int i = 0; i < PER; ++i) f[i] = i * T + tid < nranges * kTailSlots ? load_through(&slots_of[i * T + tid]) : ~(uint64_t)0;
      if (tid == 0) few_n = 0u;
      __syncthreads();
      auto add = [&](uint64_t v) __attribute__((always_inline)) {
        const uint32_t i = atomicAdd(&few_n, 1u);
        if (i < (uint32_t)kTailFew) few_all[i] = make_uint2((uint32_t)v, (uint32_t)(v >> 32) & 0x7fu);
        atomicAdd(&tail[(uint32_t)(v >> 32) & 0x7fu], 1u);
      };
#pragma unroll
      for (int i = 0; i < PER; ++i)
        if (f[i] != ~(uint64_t)0) add(f[i]);
      __syncthreads();
      const uint32_t there = same(few_n);
      if (there < cand) {  // some range has more than its places take
        __syncthreads();
        if ((uint32_t)tid < cand - there) add(load_through(&few_of[tid]));
        __syncthreads();
      }
#pragma unroll
      for (int j = 0; j < BPT; ++j) h[j] = BPT * tid < 128 ? tail[(BPT * tid + j) & 127] : 0u;
    } else {
#pragma unroll
      for (int j = 0; j < BPT / 2; ++j) {
        const uint64_t q = BPT * tid < bins ? load_through(reinterpret_cast<const uint64_t*>(dst) + BPT / 2 * tid + j) : 0ull;
        h[2 * j] = (uint32_t)q;
        h[2 * j + 1] = (uint32_t)(q >> 32);
      }
    }
    block_pick_bins<T>(st, h, stage, part, p.err);
    if (stage == 1) {
      cand = same(st.cand);
      few = cand <= (uint32_t)kTailFew;
    }
    if (stage == 0 && !spans) bound = same(st.lo);
    if (stage == 2) {
      bool reports = false;
      for (int i = 0; i < n_owned; ++i) reports = reports || owned[i] == 0;
      if (reports && tid == 0) {
        *sv.st = st1;
        if (st.level != 3u) atomicOr(p.err, kErrSequence);
      }
      if (same(st.level) != 3u) return;
      if (few) ++stage;  // (how many are kept in front of every piece is known)
    }
  }
}

template <int source>
__global__ void __launch_bounds__(64 * kTailWaves)
k_tail(SelParams p, LeaderArgs la, int row_log2) {
  __shared__ TailShared sh;
  meet_start();
  constexpr int T = 64 * kTailWaves;
  const int tid = threadIdx.x;
  // (from before this launch, or set by a block of it that has given up: see meet_wait)
  if (*p.err != 0u) return;
  if (tid == 0) sh.verdict = -1;
  if (source == kTailHist && la.partials != nullptr) {  // (every block finds, and writes, the same)
    const int best = block_take_leader(la);
    if (tid == 0) sh.verdict = best;
  }
  __syncthreads();
  SegView sv = seg_view(p, blockIdx.y, same(sh.verdict));
  sv.x = same_ptr(sv.x);
  sv.hist1 = same_ptr(sv.hist1);
  sv.hist2 = same_ptr(sv.hist2);
  sv.hseg = same_ptr(sv.hseg);
  sv.htop = same_ptr(sv.htop);
  sv.tbuf = same_ptr(sv.tbuf);
  sv.tcnt = same_ptr(sv.tcnt);
  sv.list = same_ptr(sv.list);
  sv.idx_out = same_ptr(sv.idx_out);
  sv.vals_row = same_ptr(sv.vals_row);
  sv.d.k = same(sv.d.k);
  sv.d.cap = same(sv.d.cap);
  __syncthreads();  // (verdict has been read)
  if (source == kTailSpans) {
    constexpr int PER = kMaxChunks / T;
    uint32_t m[PER], sum = 0u, total;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      m[j] = PER * tid + j < sv.d.geom.nchunks ? sv.mcount[(PER * tid + j) * kMcountLine] : 0u;
      sum += m[j];
    }
    uint32_t upto = block_prefix_incl<T>(sum, sh.part, &total) - sum;
#pragma unroll
    for (int j = 0; j < PER; ++j) {  // (chunks that are not there: `total`)
      sh.chunk_at[PER * tid + j] = upto;
      upto += m[j];
    }
    total = same(total);
    if (tid == 0) sh.chunk_at[kMaxChunks] = total;
    const uint32_t bound = same(sv.ctrl[1]);
    uint64_t limit = (uint64_t)sv.d.k + ((uint64_t)p.n >> 3);  // (k_pick_mask's rule)
    if (limit > sv.d.cap) limit = sv.d.cap;
    if (bound != kNoGuess && total >= sv.d.k && total <= limit)
      return tail_select<kTailSpans, false>(p, sv, sh, row_log2, bound, total);
    return tail_select<kTailNone, true>(p, sv, sh, row_log2, 0u, 0u);
  }
  tail_select<source, false>(p, sv, sh, row_log2, 0u, 0u);
}

// ---------------------------------------------------------------------------
// Selection from marked tiles.  Where the leader's vector is read anyway (its own pass, the leader known up front) or once
// (segments whose leader comes from the data), every segment is cut into tiles of kMarkTile elements and
//   k_guess_segs / k_guess_tiles   sample it for a lower bound on the key of its k-th largest magnitude,
//   k_mark_tiles   reads (and, with gradients, writes) the vector once: a tile's elements that reach the bound are stored in
//                  order as the tile's piece of (index, raw bits), and counted in 4095 narrow bins above the bound,
//   k_tiles_pick   finds the threshold's bin, or that the bound does not hold,
//   k_tiles_full   (only then) gives the pieces back and counts the top digits of everything,
//   k_tiles_digit  counts the next digits of the bin's keys, and per tile what lies above the bin,
//   k_tiles_count  knows the threshold and counts per tile what is kept,
//   k_tiles_out    puts a tile's kept entries where they belong.
// A tile with more marked elements than a piece takes, and every tile of a segment without a bound (too dense ones, and where
// it did not hold), has no piece: its values are in the vector, and the kernels behind the marking read them there, the waves
// of a block a part each.  The bins are so narrow that few keys share the threshold's: k_tiles_count looks only at the tiles
// that have one.  So a piece is read twice, once to count what is above the bin and once to put it out, by a wave to itself.
//   One list of all pieces instead (its writing, two digit counts and final pass 66 + 38 + 36 + 89 us for 14 M entries, and 5
// for each of three launches that had nothing to do), and for segments per-chunk histograms, which the leader's vector was
// read again for: 138 M x 4, leader known, one in ten kept 1671 us a step, now 1507, in 16 Mi buckets, one in a hundred, 1474
// / 1295, 25.6 M x 8 in 54 segments, variance rule, 642 / 622.  What values do to it, us, before / now, one in a hundred:
// 25.6 M x 2 normal 222/203, layers of 54 scales 221/215, a run of large values 250/243, sorted 377/300, all equal 610/505;
// 138 M x 2 833/769, 882/811, 955/852, 1107/901, 3144/1776; in buckets 947/783, 946/779, 973/789, 1860/1527, 2850/2339.
//   Tiles without pieces a wave each: 25.6 M x 2 with a run 280; a block of four waves each 241, but all ties 222 (four times
// the blocks add to the same digits), and 138 M in buckets 1330.
// ---------------------------------------------------------------------------
struct TileArgs {
  const uint4* map;      // [tiles] (first element, a multiple of 4; first and last + 1 of the segment's; segment), or nullptr: one segment
  const uint2* groups;   // [blocks of the kernels behind the marking] (segment, number among its blocks), or nullptr
  uint2* pieces;         // each tile's from piece_at of its first own element on
  uint32_t* held;        // [tiles] entries of the piece, or kTileOverflow
  uint32_t* marked;      // [tiles] elements that reach the bound
  // of each tile's kTileWaves parts, of which a tile with a piece has the first only:
  uint32_t* above;       // keys above the threshold's bin; then kept ones above the threshold
  uint32_t* among;       // keys in it; then those equal to the threshold
  uint32_t* slots;       // [kTileSlots] the first of those
  uint32_t* bins;        // [segments] bins_stride words apart
  int64_t bins_stride;
  uint32_t* more_bins;   // [SegDesc::bins_begin + bins_more][kHistBins]
  uint64_t* kept;        // [tiles], then [blocks] kept entries: above the threshold << 32 | at it
  uint32_t* any_full;    // set where some segment's bound does not hold
  int32_t* tile_start;   // kept entries in front of every tile of the streaming passes (two of these), or nullptr
  int32_t ntiles, ngroups;
};
// Where the piece of a tile whose own elements begin with `lo` lies, and how many entries the piece of [lo, hi) can have:
// three for sixteen elements, so that pieces lie as the tiles do, whole tiles have room for more than kMarkMax, and however
// many short segments there are takes nothing from the others (an equal share for each tile, 8.4 M elements in 250 segments
// from 500 to 200,000 long, one in ten kept: no share was large enough, 181 us to select, list kernels 93).
constexpr int kPieceOf = 16, kPieceEntries = 3;
__host__ __device__ constexpr int64_t piece_at(int64_t lo) { return lo * kPieceEntries / kPieceOf; }
__host__ __device__ constexpr uint32_t piece_room(uint32_t lo, uint32_t hi) {
  const int64_t room = piece_at(hi) - piece_at(lo);
  return room < (int64_t)kMarkMax ? (uint32_t)room : (uint32_t)kMarkMax;
}
static_assert(piece_at(kMarkTile) >= kMarkMax, "a whole tile's marks are bounded by what fits on chip");
// Up to so many tiles a block's lie apart (few in the build for tests, so that both forms run on short vectors): each wave then
// adds up what is in front of its own, which long vectors have too many tiles for.
#ifdef ARTOPK_HELD_BLOCKS
constexpr int kTilesApart = 16;
#else
constexpr int kTilesApart = 4096;
#endif
constexpr int kTileWaves = 4;  // waves, and tiles, of a block of the kernels behind the marking; and parts of a tile without a piece
constexpr int kTileSlots = 4;
constexpr uint32_t kTileOverflow = 0xffffffffu;
constexpr int kGuessLooks = 1 << 14;  // of a block of k_guess_tiles for the others, at most (some 10 ms)
// How far the threshold is known: keys [lo, lo + 2^bits), `above` of them higher, `need` of the `cand` in it kept.
// A bin of so few bits (2^7 keys at most) has its keys counted in 32 copies, 128 words apart, by 32nds of the blocks: where a
// few values are common, thousands of blocks add to them, and additions to one line of memory wait for each other (138 M x 2,
// 84 thousand values, 1650 equal ones each: 159 us for the count, now 14).
constexpr uint32_t kTileCopyBits = 7u;
struct TilePick {
  uint32_t lo, bits, above, need, cand;
};

// Bins of 4096 by rank: T threads' counts of the bins BPT t .., how many lie above them (scan), and the bin that the
// need-th largest key falls into (find; res: bin, keys above it, keys in it); all threads call them.
template <int T>
struct TileBins {
  static constexpr int BPT = kHistBins / T;
  uint32_t h[BPT];
  uint32_t above;
  __device__ __forceinline__ void scan(uint32_t* part) {
    uint32_t tot = 0u;
#pragma unroll
    for (int j = 0; j < BPT; ++j) tot += h[j];
    above = block_suffix_incl<T>(tot, part) - tot;
  }
  // false: there are not so many.  (res is free again behind it.)
  __device__ __forceinline__ bool find(uint32_t need, uint32_t* res, uint4& got) const {
    if (threadIdx.x == 0) res[0] = ~0u;
    __syncthreads();
    uint32_t upto = above;
#pragma unroll
    for (int j = BPT - 1; j >= 0; --j) {
      if (upto < need && need <= upto + h[j]) {
        res[0] = (uint32_t)(BPT * (int)threadIdx.x + j);
        res[1] = upto;
        res[2] = h[j];
      }
      upto += h[j];
    }
    __syncthreads();
    got = make_uint4(res[0], res[1], res[2], 0u);
    __syncthreads();
    return got.x != ~0u;
  }
};

// Narrows `pk` by the bits that the bins tell apart, or the counts in memory.
template <int T>
__device__ __forceinline__ void tile_take(TileBins<T>& tb, TilePick& pk, uint32_t bits, uint32_t* part, uint32_t* res,
                                          uint32_t* __restrict__ err) {
  uint4 got;
  tb.scan(part);
  if (tb.find(pk.need, res, got)) {
    pk.lo += got.x << bits;
    pk.above += got.y;
    pk.need -= got.y;
    pk.cand = got.z;
  } else if (threadIdx.x == 0) {
    atomicOr(err, kErrPick);
  }
  pk.bits = bits;
}

template <int T>
__device__ __forceinline__ void tile_narrow(TilePick& pk, const uint32_t* __restrict__ hist, uint32_t bits, uint32_t* part,
                                            uint32_t* res, uint32_t* __restrict__ err) {
  TileBins<T> tb;
  constexpr int BPT = TileBins<T>::BPT;
  static_assert(BPT % 4 == 0, "whole uint4 groups per thread");
#pragma unroll
  for (int j = 0; j < BPT / 4; ++j) {
    const uint4 q = reinterpret_cast<const uint4*>(hist)[(BPT / 4) * threadIdx.x + j];
    tb.h[4 * j + 0] = q.x;
    tb.h[4 * j + 1] = q.y;
    tb.h[4 * j + 2] = q.z;
    tb.h[4 * j + 3] = q.w;
  }
  if (pk.bits <= kTileCopyBits) {  // (the same in every thread; `part` holds T >= 128 words)
    static_assert(T >= 1 << kTileCopyBits, "a word of `part` for each bin");
    __syncthreads();
    part[threadIdx.x] = 0u;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < BPT; ++j)
      if (tb.h[j] != 0u) atomicAdd(&part[(BPT * (int)threadIdx.x + j) & ((1 << kTileCopyBits) - 1)], tb.h[j]);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < BPT; ++j) {
      const int b = BPT * (int)threadIdx.x + j;
      tb.h[j] = b < 1 << kTileCopyBits ? part[b] : 0u;
    }
    __syncthreads();
  }
  tile_take(tb, pk, bits, part, res, err);
}

// Bits below the second digit of a bin of `bits`, which takes twelve.
__device__ __forceinline__ uint32_t tile_rest(uint32_t bits) { return bits > 12u ? bits - 12u : 0u; }

// What k_tiles_pick found of the segment, and where its bound did not hold the pick from k_tiles_full's counts.
template <int T>
__device__ __forceinline__ TilePick tile_first(const SegView& sv, uint32_t* part, uint32_t* res, uint32_t* __restrict__ err) {
  const SelState st = *sv.st;
  TilePick pk{st.lo, st.pad[0], st.n_gt, st.need, st.cand};
  if (st.need_full != 0u) {
    pk = TilePick{0u, 31u, 0u, sv.d.k, 0u};
    tile_narrow<T>(pk, sv.hseg, 19u, part, res, err);
  }
  return pk;
}

// Adds the counts of T threads to `dst`, and clears them; a thread has its own.
template <int T>
__device__ __forceinline__ void tile_flush(uint32_t* lh, uint32_t* __restrict__ dst) {
#pragma unroll
  for (int i = 0; i < kHistBins / 4 / T; ++i) {
    const int b = (int)threadIdx.x + i * T;
    const uint4 q = reinterpret_cast<uint4*>(lh)[b];
    if (q.x) atomicAdd(dst + 4 * b + 0, q.x);
    if (q.y) atomicAdd(dst + 4 * b + 1, q.y);
    if (q.z) atomicAdd(dst + 4 * b + 2, q.z);
    if (q.w) atomicAdd(dst + 4 * b + 3, q.w);
    reinterpret_cast<uint4*>(lh)[b] = make_uint4(0u, 0u, 0u, 0u);
  }
}

// Where tile t of segment seg adds its bins: long segments' blocks would wait for each other at the same few hundred.
__device__ __forceinline__ uint32_t* tile_bins(const SelParams& p, const TileArgs& a, int seg, uint32_t t) {
  const SegDesc& d = p.table != nullptr ? p.table[seg] : p.one;
  const uint32_t more = (uint32_t)d.bins_more, c = t % (more + 1u);
  return c == more ? a.bins + (size_t)seg * (size_t)a.bins_stride : a.more_bins + (size_t)(d.bins_begin + (int)c) * kHistBins;
}

// Tile t: its first element (of 4 in a row), and which of the segment's it has.
__device__ __forceinline__ uint4 tile_at(const TileArgs& a, int64_t n, int64_t t) {
  if (a.map != nullptr) return a.map[t];
  const int64_t first = t * kMarkTile;
  return make_uint4((uint32_t)first, (uint32_t)first, (uint32_t)(first + kMarkTile < n ? first + kMarkTile : n), 0u);
}

// ---------------------------------------------------------------------------
// k_tile_map : TileArgs::map and groups of a segmented layout, one block per segment.  A segment's tiles start with the line
// of its first element.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
k_tile_map(const SegDesc* __restrict__ table, uint4* __restrict__ map, uint2* __restrict__ groups) {
  const SegDesc d = table[blockIdx.x];
  const int64_t line = d.e_lo & ~(int64_t)31;
  for (int t = threadIdx.x; t < d.ntiles; t += 256) {
    const int64_t first = line + (int64_t)t * kMarkTile, end = first + kMarkTile;
    map[d.tile_begin + t] = make_uint4((uint32_t)first, (uint32_t)(first < d.e_lo ? d.e_lo : first),
                                       (uint32_t)(end < d.e_hi ? end : d.e_hi), (uint32_t)blockIdx.x);
    if (t % kTileWaves == 0) groups[d.group_begin + t / kTileWaves] = make_uint2((uint32_t)blockIdx.x, (uint32_t)(t / kTileWaves));
  }
}

// ---------------------------------------------------------------------------
// k_guess_tiles : the bound of a flat vector, from `runs` runs of the sample that k_guess takes, one a thread.
// Bound by its trips to memory: the blocks count the keys' top digits, wait for each other once, pick the
// digits of three ranks (m_hi for the bound, m_mid for the sample's own threshold, m_lo for what surely lies above it), each
// block for itself, and count the second digits of the first two; the last one through picks from these.  (In two launches,
// the keys stored in between and 64 blocks of 256 threads adding to the same few hundred bins, 16.7 + 17.1 us.)
//   A block that has waited long leaves; then nobody is the last, and the vector has no bound, which costs time only.
// ---------------------------------------------------------------------------
// A block's share of a sample, from run `first` on: runs of RUN elements, run r at element at(r), RUN / 4 lanes to a run, so
// that a wave's load touches no more lines than it has to (a run a lane: twice the time).  RUN / 4 groups of four keys a
// thread, bit j of the result says whether group j is there.  GT = kGNone: xp's own keys.
template <int GT, int RUN, int T, typename At>
__device__ __forceinline__ uint32_t sample_keys(const float* __restrict__ gp, const float* __restrict__ xp, int first, int runs,
                                                At at, uint32_t (&key)[RUN]) {
  constexpr int PER = RUN / 4;
  v4f a[PER], b[PER];
  uint32_t there = 0u;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int r = first + j * (T / PER) + (int)threadIdx.x / PER;
    const int64_t e = at(r < runs ? r : runs - 1) + 4 * ((int)threadIdx.x % PER);
    if (GT != kGNone) a[j] = load4g<false, GT>(gp, e);
    b[j] = load4<false>(xp + e);
    there |= r < runs ? 1u << j : 0u;
  }
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    key[4 * j + 0] = __float_as_uint(GT != kGNone ? a[j].x + b[j].x : b[j].x) & kKeyMask;
    key[4 * j + 1] = __float_as_uint(GT != kGNone ? a[j].y + b[j].y : b[j].y) & kKeyMask;
    key[4 * j + 2] = __float_as_uint(GT != kGNone ? a[j].z + b[j].z : b[j].z) & kKeyMask;
    key[4 * j + 3] = __float_as_uint(GT != kGNone ? a[j].w + b[j].w : b[j].w) & kKeyMask;
  }
  return there;
}

// Counts the keys' top digits in lh.
template <int RUN>
__device__ __forceinline__ void sample_first(const uint32_t (&key)[RUN], uint32_t there, uint32_t* lh) {
#pragma unroll
  for (int i = 0; i < RUN; ++i)
    if ((there >> (i / 4)) & 1u) atomicAdd(&lh[key[i] >> 19], 1u);
}

// Counts the second digits of the keys with top digit `low` in lh[0], with top digit `mid` in lh[1].
template <int RUN>
__device__ __forceinline__ void sample_second(const uint32_t (&key)[RUN], uint32_t there, uint32_t low, uint32_t mid,
                                              uint32_t (*lh)[kHistBins]) {
#pragma unroll
  for (int i = 0; i < RUN; ++i) {
    const bool ok = (there >> (i / 4)) & 1u;
    if (ok && (key[i] >> 19) == low) atomicAdd(&lh[0][(key[i] >> 7) & 0xfffu], 1u);
    if (ok && (key[i] >> 19) == mid) atomicAdd(&lh[1][(key[i] >> 7) & 0xfffu], 1u);
  }
}

constexpr int kGuessThreads = 512;
template <int GT>
__global__ void __launch_bounds__(kGuessThreads)
k_guess_tiles(const float* __restrict__ gp, const float* __restrict__ rp, uint32_t* __restrict__ slot, int runs,
              int64_t stride, uint32_t m_hi, uint32_t m_mid, uint32_t m_lo, uint32_t* __restrict__ info) {
  constexpr int T = kGuessThreads;
  __shared__ __attribute__((aligned(16))) uint32_t lh[2][kHistBins];
  __shared__ uint32_t part[T / 64];
  __shared__ uint32_t res[4];
  __shared__ int sh;
  const int tid = threadIdx.x;
  meet_start();
  uint32_t* __restrict__ ctrl = slot + kSlotCtrl;
  uint32_t key[kGuessRun];
  const uint32_t there = sample_keys<GT, kGuessRun, T>(
      gp, rp, (int)blockIdx.x * T, runs, [&](int r) { return ((int64_t)r * stride) & ~(int64_t)(kGuessRun - 1); }, key);
  for (int i = tid; i < 2 * kHistBins / 4; i += T) reinterpret_cast<uint4*>(lh[0])[i] = make_uint4(0u, 0u, 0u, 0u);
  if (tid == 0) sh = 0;
  __syncthreads();
  sample_first(key, there, lh[0]);
  __syncthreads();
  tile_flush<T>(lh[0], slot + (blockIdx.x % 2u == 0u ? kSlotGuessHist : kGuessOddAt));
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (what this wave has added is there: see meet_arrive)
  __syncthreads();
  if (tid == 0) {
    __hip_atomic_fetch_add(&ctrl[0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int looks = meet_limit() < kGuessLooks ? meet_limit() : kGuessLooks;
    for (int i = 0; i < looks && sh == 0; ++i) sh = load_through(&ctrl[0]) == gridDim.x ? 1 : 0;
  }
  __syncthreads();
  if (sh == 0) return;
  TileBins<T> tb;
  auto read = [&](const uint32_t* hist, const uint32_t* more) __attribute__((always_inline)) {
    uint64_t q[TileBins<T>::BPT / 2], m[TileBins<T>::BPT / 2];
#pragma unroll
    for (int j = 0; j < TileBins<T>::BPT / 2; ++j) {
      q[j] = load_through(reinterpret_cast<const uint64_t*>(hist) + TileBins<T>::BPT / 2 * tid + j);
      m[j] = more != nullptr ? load_through(reinterpret_cast<const uint64_t*>(more) + TileBins<T>::BPT / 2 * tid + j) : 0ull;
    }
#pragma unroll
    for (int j = 0; j < TileBins<T>::BPT / 2; ++j) {
      tb.h[2 * j] = (uint32_t)q[j] + (uint32_t)m[j];
      tb.h[2 * j + 1] = (uint32_t)(q[j] >> 32) + (uint32_t)(m[j] >> 32);
    }
    tb.scan(part);
  };
  uint4 low, mid, top, low2, mid2;
  read(slot + kSlotGuessHist, slot + kGuessOddAt);
  if (!tb.find(m_hi, res, low) || low.x >= 0xff0u) return;  // (bounds beyond infinity's digit: none)
  tb.find(m_mid, res, mid);
  tb.find(m_lo, res, top);
  sample_second(key, there, low.x, mid.x, lh);
  __syncthreads();
  tile_flush<T>(lh[0], slot + kGuessLowAt);
  tile_flush<T>(lh[1], slot + kGuessMidAt);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) sh = __hip_atomic_fetch_add(&ctrl[2], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1 ? 1 : 0;
  __syncthreads();
  if (sh == 0) return;
  read(slot + kGuessLowAt, nullptr);
  const bool ok = tb.find(m_hi - low.y, res, low2);
  read(slot + kGuessMidAt, nullptr);
  const bool ok_mid = tb.find(m_mid - mid.y, res, mid2);
  if (tid == 0) tile_info(info, (low.x << 19) | (ok ? low2.x << 7 : 0u), (mid.x << 19) | (ok_mid ? mid2.x << 7 : 0u), top.x);
}

// ---------------------------------------------------------------------------
// k_guess_segs : the bounds of a segmented selection, one block of 1024 threads per segment.  Up to 1024 runs of 32
// elements, a line of memory each, are sampled, one a thread; the bound's rank is the sample's share of k and six standard deviations, widened by
// how much the runs' counts differ from each other (values that lie together are worth fewer draws).  Bound by loading
// them (a block's lines come at about 0.4 a ns).  Segments too dense for pieces get no bound.
// ---------------------------------------------------------------------------
constexpr int kSegRun = 32, kSegRuns = 1024;
// What is sampled of the segment [lo, hi): its lines from `first` on, `runs` of them, all of a short one's (but for a few
// elements at its ends: the bound is then exact).
struct SegSample {
  int64_t first, runs;
  bool whole;
  float expect, chance;  // of its k largest in the sample, and six standard deviations of draws that know nothing of each other
  __host__ __device__ SegSample(int64_t lo, int64_t hi, int64_t k) {
    const int64_t len = hi - lo;
    first = (lo + kSegRun - 1) / kSegRun * kSegRun;
    whole = len <= kSegRuns * kSegRun;
    runs = whole ? (hi - first) / kSegRun : len / (4 * kSegRun);
    if (runs > kSegRuns) runs = kSegRuns;
    expect = whole ? (float)k : (float)k * elements() / (float)len;
    chance = whole ? 0.0f : 6.0f * sqrtf(expect) + 8.0f;
  }
  __host__ __device__ float elements() const { return (float)(runs * kSegRun); }
  // Whether a piece holds what a tile is expected to mark, and six standard deviations where it shares the marks with other
  // tiles: up to about one in seven kept.
  __host__ __device__ bool has_pieces(int64_t lo, int64_t hi, int ntiles) const {
    if (runs < 1) return false;
    const float len = (float)(hi - lo), tile = len < (float)kMarkTile ? len : (float)kMarkTile;
    const float marks = (expect + chance) / (whole ? len : elements()) * tile;
    return marks + (ntiles > 1 ? 6.0f * sqrtf(marks) : 0.0f) <=
           (float)piece_room((uint32_t)lo, (uint32_t)(ntiles > 1 ? lo + kMarkTile : hi));
  }
};

template <int GT>
__global__ void __launch_bounds__(kSegRuns)
k_guess_segs(SelParams p, PtrTable g) {
  constexpr int T = kSegRuns;
  __shared__ __attribute__((aligned(16))) uint32_t lh[2][kHistBins];
  __shared__ uint32_t part[T / 64];
  __shared__ uint32_t res[4];
  __shared__ uint64_t wsum[T / 64];
  const int seg = blockIdx.x, tid = threadIdx.x;
  const SegView sv = seg_view(p, seg);
  const int64_t len = sv.d.e_hi - sv.d.e_lo;
  const int64_t k = sv.d.k;
  const SegSample of(sv.d.e_lo, sv.d.e_hi, k);
  if (!of.has_pieces(sv.d.e_lo, sv.d.e_hi, sv.d.ntiles)) return;  // (`info` has been cleared)
  const bool whole = of.whole;
  const int64_t runs = of.runs, e_first = of.first;
  const float sample = of.elements(), expect = of.expect;
  const int64_t stride = whole ? kSegRun : len / runs;
  uint32_t key[kSegRun];
  const uint32_t there = sample_keys<GT, kSegRun, T>(
      g.p[0], sv.x, 0, (int)runs,
      [&](int r) { return e_first + ((r * stride) & ~(int64_t)(kSegRun - 1)); },  // (the last one ends in front of the segment's end)
      key);
  for (int i = tid; i < 2 * kHistBins / 4; i += T) reinterpret_cast<uint4*>(lh[0])[i] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  sample_first(key, there, lh[0]);
  __syncthreads();
  TileBins<T> tb;
  auto read = [&](int which) __attribute__((always_inline)) {
    const uint4 q = reinterpret_cast<const uint4*>(lh[which])[tid];
    tb.h[0] = q.x;
    tb.h[1] = q.y;
    tb.h[2] = q.z;
    tb.h[3] = q.w;
    tb.scan(part);
  };
  const uint32_t m_mid = (uint32_t)fmaxf(1.0f, expect + 0.5f);
  uint4 low, mid, top, low2, mid2;
  read(0);
  reinterpret_cast<uint4*>(lh[0])[tid] = make_uint4(0u, 0u, 0u, 0u);
  if (!tb.find(m_mid, res, mid)) return;
  // how the runs' counts of keys that reach that digit vary, against draws that know nothing of each other
  uint32_t c1 = 0u, c2 = 0u;
#pragma unroll
  for (int j = 0; j < kSegRun / 4; ++j) {
    uint32_t c = 0u;
#pragma unroll
    for (int e = 0; e < 4; ++e) c += ((there >> j) & 1u) && (key[4 * j + e] >> 19) >= mid.x ? 1u : 0u;
    c1 += c;
#pragma unroll
    for (int off = 1; off < kSegRun / 4; off <<= 1) c += __shfl_xor(c, off, 64);
    c2 += tid % (kSegRun / 4) == 0 ? c * c : 0u;
  }
  const uint64_t both = wave_allsum_u64(((uint64_t)c1 << 32) | c2);
  if ((tid & 63) == 0) wsum[tid >> 6] = both;
  __syncthreads();
  uint64_t all = 0ull;
#pragma unroll
  for (int i = 0; i < T / 64; ++i) all += wsum[i];
  const float s1 = (float)(uint32_t)(all >> 32), s2 = (float)(uint32_t)all;
  const float wide = fmaxf(1.0f, (s2 - s1 * s1 / (float)runs) / fmaxf(1.0f, s1));
  const float margin = whole ? 0.0f : 6.0f * sqrtf(expect * wide) + 8.0f;
  if (expect + margin > sample) return;
  const uint32_t m_hi = whole ? (uint32_t)k : (uint32_t)ceilf(expect + margin);
  const float less = whole ? 64.0f : margin;  // (as many may be missing)
  if (!tb.find(m_hi, res, low) || low.x >= 0xff0u) return;  // (bounds beyond infinity's digit: none)
  tb.find((uint32_t)fmaxf(1.0f, expect - less), res, top);
  sample_second(key, there, low.x, mid.x, lh);
  __syncthreads();
  read(0);
  const bool ok = tb.find(m_hi - low.y, res, low2);
  read(1);
  const bool ok_mid = tb.find(m_mid - mid.y, res, mid2);
  if (tid == 0)
    tile_info(p.zero_base + (size_t)seg * kSegWords + kTileInfo, (low.x << 19) | (ok ? low2.x << 7 : 0u),
              (mid.x << 19) | (ok_mid ? mid2.x << 7 : 0u), top.x);
}

// ---------------------------------------------------------------------------
// k_mark_tiles : acc = g + residual (in place over residual; GT = kGNone: the vector is only read), and every tile's marked
// elements as its piece and in the segment's bins.  grid = blocks striding over the tiles.  Bound by memory: 138 M elements,
// one in a hundred kept, 273 us (6.1 TB/s), one in ten 318 (5.6; with blocks of twice the threads and tile, of which one fits
// a compute unit instead of two, 348, so that nothing is loaded while a tile's marks are ranked); where few tiles are only
// read, by instructions (25.6 M 38 us, of which a block ranks its marks for a third).  An element is marked if not |x| < bound (a NaN is).
// Marked elements from the sample's own estimate of the threshold on are stored as +0.0 at once: nearly all of them are
// kept, nearly none of those below, and k_tiles_out puts the others right.
// ---------------------------------------------------------------------------
template <bool NT, int GT>
__global__ void __launch_bounds__(kMarkThreads, GT == kGNone ? 8 : 4)
k_mark_tiles(SelParams p, TileArgs a, const float* __restrict__ gp, float* __restrict__ rp) {
  constexpr int T = kMarkThreads, U = 8, WAVES = T / 64;
  static_assert(T * U * 4 == kMarkTile && WAVES * U == 64, "a tile a block, and a lane for every row's count");
  __shared__ uint32_t wcnt[WAVES * U];  // the tile's row counts, row-major
  __shared__ uint2 stage[kMarkMax];
  __shared__ __attribute__((aligned(16))) uint32_t lh[kHistBins];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (GT == kGNone) rp = p.tab.p[p.one.vec >= 0 ? p.one.vec : *p.leader_dev];
#pragma unroll
  for (int i = 0; i < kHistBins / 4 / T; ++i) reinterpret_cast<uint4*>(lh)[tid + i * T] = make_uint4(0u, 0u, 0u, 0u);
  for (int64_t ti = blockIdx.x; ti < a.ntiles; ti += gridDim.x) {
    const uint4 at = tile_at(a, p.n, ti);
    const int seg = (int)__builtin_amdgcn_readfirstlane(at.w);
    const uint32_t first = __builtin_amdgcn_readfirstlane(at.x), lo = __builtin_amdgcn_readfirstlane(at.y);
    const uint32_t hi = __builtin_amdgcn_readfirstlane(at.z);
    const uint32_t* __restrict__ info = p.zero_base + (size_t)seg * kSegWords + kTileInfo;
    const uint32_t bound = info[kTileBound], shift = info[kTileShift], zero = info[kTileZero];
    const float gf = __uint_as_float(bound), zf = __uint_as_float(zero);
    const uint32_t q0 = (first >> 2) + (uint32_t)tid;
    uint32_t own = 0u;       // bit 4 u + e: element e of this lane's group in row u is marked
    uint32_t rows_cnt = 0u;  // lane u < U: marks of the wave's row u
    uint32_t zeroed = 0u;    // as own: stored as +0.0
    uint32_t bits[U][4];
    // FULL: the whole tile is the segment's, so nothing is predicated.
    auto load = [&](auto full_tag) {
      constexpr bool FULL = decltype(full_tag)::value;
      const uint32_t w_lo = (lo + 3u) >> 2, w_hi = hi >> 2;  // whole groups
      v4f x[U], b[U];
      if (FULL || w_lo < w_hi) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          // (groups outside re-read the nearest one, unused: no branch between the loads)
          const uint32_t q = q0 + (uint32_t)(u * T);
          const uint32_t ql = FULL ? q : (q < w_lo ? w_lo : (q < w_hi ? q : w_hi - 1u));
          if (GT != kGNone) x[u] = load4g<NT, GT>(gp, 4 * (int64_t)ql);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {  // (one array after the other: see k_pass_mark)
          const uint32_t q = q0 + (uint32_t)(u * T);
          const uint32_t ql = FULL ? q : (q < w_lo ? w_lo : (q < w_hi ? q : w_hi - 1u));
          b[u] = load4<NT>(rp + 4 * (int64_t)ql);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t q = q0 + (uint32_t)(u * T);
        uint32_t there = 0xfu;  // the group's elements that are the tile's
        if (!FULL) {
          there = 0u;
#pragma unroll
          for (uint32_t e = 0u; e < 4u; ++e) there |= (4u * q + e >= lo && 4u * q + e < hi) ? 1u << e : 0u;
        }
        v4f v = {0.f, 0.f, 0.f, 0.f};
        if (FULL || there == 0xfu) {
          v = b[u];
          if (GT != kGNone) {
            v.x = x[u].x + b[u].x;
            v.y = x[u].y + b[u].y;
            v.z = x[u].z + b[u].z;
            v.w = x[u].w + b[u].w;
          }
        } else if (there != 0u) {
          float s[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (uint32_t e = 0u; e < 4u; ++e)
            if ((there >> e) & 1u) {
              s[e] = rp[4 * (int64_t)q + e];
              if (GT != kGNone) s[e] = load1g<GT>(gp, 4 * (int64_t)q + e) + s[e];
            }
          v = v4f{s[0], s[1], s[2], s[3]};
        }
        const bool h0 = (FULL || (there & 1u)) && !(__builtin_fabsf(v.x) < gf);
        const bool h1 = (FULL || (there & 2u)) && !(__builtin_fabsf(v.y) < gf);
        const bool h2 = (FULL || (there & 4u)) && !(__builtin_fabsf(v.z) < gf);
        const bool h3 = (FULL || (there & 8u)) && !(__builtin_fabsf(v.w) < gf);
        const uint32_t row = (uint32_t)(__popcll(__ballot(h0)) + __popcll(__ballot(h1)) + __popcll(__ballot(h2)) + __popcll(__ballot(h3)));
        own |= ((h0 ? 1u : 0u) | (h1 ? 2u : 0u) | (h2 ? 4u : 0u) | (h3 ? 8u : 0u)) << (4 * u);
        rows_cnt = lane == u ? row : rows_cnt;
        bits[u][0] = __float_as_uint(v.x);
        bits[u][1] = __float_as_uint(v.y);
        bits[u][2] = __float_as_uint(v.z);
        bits[u][3] = __float_as_uint(v.w);
        if (GT != kGNone) {
          v4f z = v;
          uint32_t zs = 0u;
          if (bound != 0u) {
            const bool z0 = h0 && !(__builtin_fabsf(v.x) < zf), z1 = h1 && !(__builtin_fabsf(v.y) < zf);
            const bool z2 = h2 && !(__builtin_fabsf(v.z) < zf), z3 = h3 && !(__builtin_fabsf(v.w) < zf);
            z.x = z0 ? 0.0f : v.x;
            z.y = z1 ? 0.0f : v.y;
            z.z = z2 ? 0.0f : v.z;
            z.w = z3 ? 0.0f : v.w;
            zs = (z0 ? 1u : 0u) | (z1 ? 2u : 0u) | (z2 ? 4u : 0u) | (z3 ? 8u : 0u);
          }
          zeroed |= zs << (4 * u);
          if (FULL || there == 0xfu) {
            store4<NT>(rp + 4 * (int64_t)q, z);
          } else if (there != 0u) {
            const float s[4] = {z.x, z.y, z.z, z.w};
#pragma unroll
            for (uint32_t e = 0u; e < 4u; ++e)
              if ((there >> e) & 1u) rp[4 * (int64_t)q + e] = s[e];
          }
        }
      }
    };
    if (lo == first && hi == first + (uint32_t)kMarkTile)
      load(std::true_type{});
    else
      load(std::false_type{});
    if (bound == 0u) {  // no bound: every element's top digit is counted, and there is no piece
      __syncthreads();  // (the tile before has cleared the counts)
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if ((own >> (4 * u + e)) & 1u) atomicAdd(&lh[(bits[u][e] & kKeyMask) >> 19], 1u);
      if (tid == 0) {
        a.held[ti] = kTileOverflow;
        a.marked[ti] = hi - lo;
      }
      __syncthreads();
    } else {
      // rank the tile's marks: element order is row-major, row = 8 u + wave, then lane, then e
      if (lane < U) wcnt[lane * WAVES + wave] = rows_cnt;
      __syncthreads();
      const uint32_t c0 = wcnt[lane];  // (every wave scans the counts itself)
      const uint32_t s0 = wave_incl_scan(c0);
      const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)s0, 63);
      const bool fits = total <= piece_room(lo, hi);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        // marks in the rows before this wave's row u
        const uint32_t before = (uint32_t)__builtin_amdgcn_readlane((int)(s0 - c0), u * WAVES + wave);
        const uint64_t b0 = __ballot((own >> (4 * u + 0)) & 1u), b1 = __ballot((own >> (4 * u + 1)) & 1u);
        const uint64_t b2 = __ballot((own >> (4 * u + 2)) & 1u), b3 = __ballot((own >> (4 * u + 3)) & 1u);
        if (((own >> (4 * u)) & 0xfu) != 0u) {
          uint32_t pos = before + popc_lt(b0) + popc_lt(b1) + popc_lt(b2) + popc_lt(b3);
          const uint32_t j0 = 4u * (q0 + (uint32_t)(u * T));
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if ((own >> (4 * u + e)) & 1u) {
              const uint32_t bin = ((bits[u][e] & kKeyMask) - bound) >> shift;
              if (bin < (uint32_t)kTileBins) atomicAdd(&lh[bin], 1u);
              if (fits) stage[pos] = make_uint2(j0 + (uint32_t)e, bits[u][e]);
              ++pos;
            }
          }
          if (GT != kGNone && !fits && ((zeroed >> (4 * u)) & 0xfu) != 0u) {  // rare: the values go back into the vector
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if ((zeroed >> (4 * u + e)) & 1u) rp[j0 + (uint32_t)e] = __uint_as_float(bits[u][e]);
          }
        }
      }
      __syncthreads();
      if (fits) {
        uint2* __restrict__ dst = a.pieces + piece_at(lo);
        for (uint32_t i = (uint32_t)tid; i < total; i += T) dst[i] = stage[i];
      }
      if (tid == 0) {
        a.held[ti] = fits ? total : kTileOverflow;
        a.marked[ti] = total;
      }
    }
    // (the next tile counts behind its first barrier)
    tile_flush<T>(lh, tile_bins(p, a, seg, (uint32_t)ti));
  }
}

// ---------------------------------------------------------------------------
// k_tiles_pick : one block of 1024 threads per segment: the threshold's bin.  A bound that fewer than k keys reach, or more
// than k + n/8, or below which all bins lie, does not hold (need_full; the segment's own histogram is zero then).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(1024)
k_tiles_pick(SelParams p, TileArgs a) {
  constexpr int T = 1024;
  __shared__ uint32_t part[T];
  __shared__ uint32_t res[4];
  __shared__ uint64_t wsum[T / 64];
  const int seg = blockIdx.x, tid = threadIdx.x;
  const SegView sv = seg_view(p, seg);
  const uint32_t* __restrict__ info = p.zero_base + (size_t)seg * kSegWords + kTileInfo;
  const uint32_t bound = info[kTileBound], shift = bound != 0u ? info[kTileShift] : 19u;
  uint32_t* __restrict__ bins = a.bins + (size_t)seg * (size_t)a.bins_stride;
  TileBins<T> tb;
#pragma unroll
  for (int j = 0; j < 4; ++j) tb.h[j] = 0u;
  const uint4 own = reinterpret_cast<const uint4*>(bins)[tid];
  for (int r0 = 0; r0 < sv.d.bins_more; r0 += 4) {  // four copies in flight
    uint4 q[4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
      q[r] = reinterpret_cast<const uint4*>(a.more_bins +
                                            (size_t)(sv.d.bins_begin + (r0 + r < sv.d.bins_more ? r0 + r : r0)) * kHistBins)[tid];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if (r0 + r < sv.d.bins_more) {
        tb.h[0] += q[r].x;
        tb.h[1] += q[r].y;
        tb.h[2] += q[r].z;
        tb.h[3] += q[r].w;
      }
    }
  }
  tb.h[0] += own.x;
  tb.h[1] += own.y;
  tb.h[2] += own.z;
  tb.h[3] += own.w;
  uint64_t marks = 0u;
  for (int t = tid; t < sv.d.ntiles; t += 8 * T) {  // eight tiles' in flight
    uint32_t m[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) m[u] = a.marked[sv.d.tile_begin + (t + u * T < sv.d.ntiles ? t + u * T : t)];
#pragma unroll
    for (int u = 0; u < 8; ++u) marks += t + u * T < sv.d.ntiles ? m[u] : 0u;
  }
  const uint64_t binned = (uint64_t)tb.h[0] + tb.h[1] + tb.h[2] + tb.h[3];
  const uint64_t both = wave_allsum_u64((marks << 32) | binned);  // (both are below 2^31)
  if ((tid & 63) == 0) wsum[tid >> 6] = both;
  __syncthreads();
  uint64_t all = 0u;
#pragma unroll
  for (int i = 0; i < T / 64; ++i) all += wsum[i];
  const uint32_t total = (uint32_t)(all >> 32), high = bound == 0u ? 0u : total - (uint32_t)all;  // above all bins
  const uint32_t k = sv.d.k;
  uint64_t limit = (uint64_t)k + ((uint64_t)(sv.d.e_hi - sv.d.e_lo) >> 3);
  if (limit > sv.d.cap) limit = sv.d.cap;
  const bool holds = bound == 0u || (total >= k && total <= limit && high < k);
  SelState st{};
  if (holds) {
    uint4 got;
    tb.scan(part);
    if (!tb.find(k - high, res, got)) {
      if (tid == 0) atomicOr(p.err, kErrPick);
      return;
    }
    st.lo = bound + (got.x << shift);
    st.hi = st.lo + ((1u << shift) - 1u);
    st.n_gt = high + got.y;
    st.need = k - st.n_gt;
    st.cand = got.z;
    st.level = 1u;
    st.compact_level = bound != 0u || fits_list(st, sv.d.cap) ? 1u : 0u;
    st.list_count = bound != 0u ? total : st.compact_level ? st.n_gt + st.cand : 0u;
    st.use_mask = bound != 0u ? 1u : 0u;
    st.list_lo = bound;
    st.pad[0] = shift;
  } else {
    st.need_full = 1u;
    if (bins == sv.hseg) reinterpret_cast<uint4*>(bins)[tid] = make_uint4(0u, 0u, 0u, 0u);
    if (tid == 0) *a.any_full = 1u;
  }
  if (tid == 0) *sv.st = st;
}

// ---------------------------------------------------------------------------
// k_tiles_full : for segments whose bound does not hold: the marked elements get their values back, and the segment's own
// histogram the top digits of all keys.  Blocks stride over the tiles.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(kMarkThreads)
k_tiles_full(SelParams p, TileArgs a) {
  constexpr int T = kMarkThreads, U = 8;
  if (*a.any_full == 0u) return;
  __shared__ __attribute__((aligned(16))) uint32_t lh[kHistBins];
  const int tid = threadIdx.x;
#pragma unroll
  for (int i = 0; i < kHistBins / 4 / T; ++i) reinterpret_cast<uint4*>(lh)[tid + i * T] = make_uint4(0u, 0u, 0u, 0u);
  for (int64_t ti = blockIdx.x; ti < a.ntiles; ti += gridDim.x) {
    const uint4 at = tile_at(a, p.n, ti);
    const SegView sv = seg_view(p, (int)at.w);
    if (sv.st->need_full == 0u) continue;  // (the same in every thread)
    const uint32_t lo = at.y, hi = at.z, held = a.held[ti];
    const uint32_t zero = p.zero_base[(size_t)at.w * kSegWords + kTileInfo + kTileZero];
    if (p.zero_vec != nullptr && held != kTileOverflow) {
      const uint2* __restrict__ piece = a.pieces + piece_at(lo);
      for (uint32_t i = (uint32_t)tid; i < held; i += T) {
        const uint2 ent = piece[i];
        if ((ent.y & kKeyMask) >= zero && ent.x >= lo && ent.x < hi) p.zero_vec[ent.x] = __uint_as_float(ent.y);
      }
    }
    __threadfence_block();
    __syncthreads();
    if (tid == 0) a.held[ti] = kTileOverflow;
    const uint32_t w_lo = (lo + 3u) >> 2, w_hi = hi >> 2;
    auto count = [&](uint32_t raw) { wave_count(lh, (raw & kKeyMask) >> 19); };
    if (w_lo < w_hi) {
      uint4 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t q = w_lo + (uint32_t)(tid + u * T);
        v[u] = *reinterpret_cast<const uint4*>(sv.x + 4 * (int64_t)(q < w_hi ? q : w_hi - 1u));
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (w_lo + (uint32_t)(tid + u * T) < w_hi) {
          count(v[u].x);
          count(v[u].y);
          count(v[u].z);
          count(v[u].w);
        }
      }
    }
    // the elements outside whole groups: at most three on either side
    const uint32_t front = w_lo < w_hi ? 4u * w_lo - lo : hi - lo, back = w_lo < w_hi ? hi - 4u * w_hi : 0u;
    if ((uint32_t)tid < front) count(__float_as_uint(sv.x[lo + (uint32_t)tid]));
    if ((uint32_t)tid < back) count(__float_as_uint(sv.x[4 * (int64_t)w_hi + tid]));
    __syncthreads();
    tile_flush<T>(lh, sv.hseg);
    __syncthreads();
  }
}

// The entries of tile `at`: `piece`'s, `held` of them, in rows of 64 (row1(entry, whether it is there)), or where there is none
// those of the tile's part `part` from the vector, in rows of 256, four in a row a lane's (row4(raw bits, the first one's
// element, which of them are there)), in order.  The 64 lanes of a wave call it.
template <typename Row1, typename Row4>
__device__ __forceinline__ void tile_rows(const uint2* __restrict__ piece, const float* x, uint32_t held, int part, const uint4 at,
                                          Row1 row1, Row4 row4) {
  const uint32_t lane = lane_id();
  if (held != kTileOverflow) {
#pragma unroll 1
    for (uint32_t r0 = 0u; r0 < held; r0 += 512u) {  // eight rows in flight
      uint2 ent[8];
#pragma unroll
      for (uint32_t u = 0u; u < 8u; ++u) {
        const uint32_t i = r0 + 64u * u + lane;
        ent[u] = piece[i < held ? i : held - 1u];
      }
#pragma unroll
      for (uint32_t u = 0u; u < 8u; ++u)
        if (r0 + 64u * u < held) row1(ent[u], r0 + 64u * u + lane < held);
    }
    return;
  }
  constexpr uint32_t PART = kMarkTile / kTileWaves;
  const uint32_t first = __builtin_amdgcn_readfirstlane(at.x) + (uint32_t)part * PART;
  uint32_t lo = __builtin_amdgcn_readfirstlane(at.y), hi = __builtin_amdgcn_readfirstlane(at.z);
  if (lo < first) lo = first;
  if (hi > first + PART) hi = first + PART;
  if (lo == first && hi == first + PART) {
    const uint4* __restrict__ from = reinterpret_cast<const uint4*>(x + first) + lane;
    constexpr int ROWS = (int)PART / 256;
    uint4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = from[64 * u];
#pragma unroll 1
    for (int r0 = 0; r0 < ROWS; r0 += 4) {  // the next four rows' loads in front of these rows' work
      uint4 w[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) w[u] = from[64 * (r0 + 4 < ROWS ? r0 + 4 + u : u)];
#pragma unroll
      for (int u = 0; u < 4; ++u) row4(v[u], first + 256u * (uint32_t)(r0 + u) + 4u * lane, 0xfu);
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = w[u];
    }
    return;
  }
  const uint32_t w_lo = (lo + 3u) >> 2, w_hi = hi >> 2;
#pragma unroll 1
  for (uint32_t q0 = first >> 2; 4u * q0 < hi; q0 += 256u) {
    uint4 v[4];
#pragma unroll
    for (uint32_t u = 0u; u < 4u; ++u) {
      const uint32_t q = q0 + 64u * u + lane;
      v[u] = make_uint4(0u, 0u, 0u, 0u);
      if (q >= w_lo && q < w_hi) {
        v[u] = *reinterpret_cast<const uint4*>(x + 4 * (int64_t)q);
      } else {  // at most one group on either side
        if (4u * q + 0u >= lo && 4u * q + 0u < hi) v[u].x = __float_as_uint(x[4 * (int64_t)q + 0]);
        if (4u * q + 1u >= lo && 4u * q + 1u < hi) v[u].y = __float_as_uint(x[4 * (int64_t)q + 1]);
        if (4u * q + 2u >= lo && 4u * q + 2u < hi) v[u].z = __float_as_uint(x[4 * (int64_t)q + 2]);
        if (4u * q + 3u >= lo && 4u * q + 3u < hi) v[u].w = __float_as_uint(x[4 * (int64_t)q + 3]);
      }
    }
#pragma unroll 1
    for (uint32_t u = 0u; u < 4u; ++u) {
      const uint32_t q = q0 + 64u * u + lane;
      uint32_t there = 0u;
#pragma unroll
      for (uint32_t e = 0u; e < 4u; ++e) there |= (4u * q + e >= lo && 4u * q + e < hi) ? 1u << e : 0u;
      if (4u * (q0 + 64u * u) < hi) row4(v[0], 4u * q, there);
      v[0] = v[1];
      v[1] = v[2];
      v[2] = v[3];
    }
  }
}

// What a block of k_tiles_digit, k_tiles_count or k_tiles_out has: kTileWaves tiles of a segment, side by side, or (APART)
// as many blocks apart as the segment has, so that a few blocks do not get all the tiles without pieces where large values lie
// together.  A wave first takes its own tile's piece, then its part of each tile of the block that has none.
template <bool APART>
struct TileGroup {
  int seg, number, blocks, ntiles;
  int64_t begin;
  const uint2* piece;  // of the wave's own tile
  uint32_t own;   // its entries
  uint32_t open;  // bit i: the block's i-th tile has none
  __device__ __forceinline__ TileGroup(const SelParams& p, const TileArgs& a, int wave) {
    seg = 0;
    number = (int)blockIdx.x;
    if (a.groups != nullptr) {
      const uint2 g = a.groups[blockIdx.x];
      seg = (int)__builtin_amdgcn_readfirstlane(g.x);
      number = (int)__builtin_amdgcn_readfirstlane(g.y);
    }
    const SegDesc& d = p.table != nullptr ? p.table[seg] : p.one;
    ntiles = d.ntiles;
    begin = d.tile_begin;
    blocks = (ntiles + kTileWaves - 1) / kTileWaves;
    const int i = (int)lane_id() & (kTileWaves - 1);
    const int64_t t = begin + (tile(i) < ntiles ? tile(i) : 0);
    const uint32_t held = a.held[t], lo = tile_at(a, p.n, t).y;
    piece = a.pieces + piece_at((uint32_t)__builtin_amdgcn_readlane((int)lo, wave));
    own = (uint32_t)__builtin_amdgcn_readlane((int)held, wave);
    open = (uint32_t)__ballot(tile(i) < ntiles && held == kTileOverflow) & ((1u << kTileWaves) - 1u);
  }
  // the segment's tile that is the block's i-th; ntiles or more where there is none
  __device__ __forceinline__ int tile(int i) const { return APART ? number + i * blocks : number * kTileWaves + i; }
  // job(the block's tile, the part of it) for whatever wave `wave` has to do, in some order
  template <typename Job>
  __device__ __forceinline__ void each(int wave, Job job) const {
#pragma unroll 1
    for (int n = 0; n <= kTileWaves; ++n) {
      const int i = n == 0 ? wave : n - 1;
      if (tile(i) < ntiles && (n == 0) != (((open >> i) & 1u) != 0u)) job(i, n == 0 ? own : kTileOverflow, n == 0 ? 0 : wave);
    }
  }
};

// ---------------------------------------------------------------------------
// k_tiles_digit : counts the next digits of the keys in the threshold's bin (LEVEL 1: twelve bits, and per tile how many lie
// above the bin, how many in it, and the first few of these; LEVEL 2: the up to seven bits that are left where the bin was
// as wide as a top digit).
// ---------------------------------------------------------------------------
template <int LEVEL, bool APART>
__global__ void __launch_bounds__(64 * kTileWaves)
k_tiles_digit(SelParams p, TileArgs a) {
  constexpr int T = 64 * kTileWaves;
  __shared__ __attribute__((aligned(16))) uint32_t lh[kHistBins];
  __shared__ uint32_t part[T];
  __shared__ uint32_t res[4];
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t lane = lane_id();
  if (*p.err != 0u) return;
  const TileGroup<APART> tg(p, a, wave);
  const SegView sv = seg_view(p, tg.seg);
  if (LEVEL == 2 && sv.st->need_full == 0u && tile_rest(sv.st->pad[0]) == 0u) return;
#pragma unroll
  for (int i = 0; i < kHistBins / 4 / T; ++i) reinterpret_cast<uint4*>(lh)[tid + i * T] = make_uint4(0u, 0u, 0u, 0u);
  TilePick pk = tile_first<T>(sv, part, res, p.err);
  if (LEVEL == 1 && tg.number == 0 && tid == 0 && sv.st->need_full != 0u) {  // what select_info reports
    SelState st{};
    st.n_gt = pk.above;
    st.cand = pk.cand;
    const bool fits = fits_list(st, sv.d.cap);
    sv.st->list_count = fits ? pk.above + pk.cand : 0u;
    sv.st->compact_level = fits ? 1u : 0u;
  }
  if (LEVEL == 2) tile_narrow<T>(pk, sv.hist1, tile_rest(pk.bits), part, res, p.err);
  __syncthreads();
  const uint32_t klo = pk.lo, khi = pk.lo + ((1u << pk.bits) - 1u), rest = LEVEL == 2 ? 0u : tile_rest(pk.bits);
  const uint32_t width = khi - klo;
  const uint32_t copy = LEVEL == 1 && pk.bits <= kTileCopyBits ? (blockIdx.x % (kHistBins >> kTileCopyBits)) << kTileCopyBits : 0u;
  tg.each(wave, [&](int i, uint32_t held, int q) __attribute__((always_inline)) {
    const int64_t t = tg.begin + tg.tile(i), tp = t * kTileWaves + q;
    if (LEVEL == 2 && a.among[tp] == 0u) return;
    uint32_t up = 0u, in = 0u;  // a lane's own; the wave's
    auto middle = [&](uint32_t kk, bool mid) __attribute__((always_inline)) {
      const uint64_t m = __ballot(mid);
      if (mid) {
        wave_count(lh, copy + ((kk - klo) >> rest));
        const uint32_t at = in + popc_lt(m);
        if (LEVEL == 1 && at < (uint32_t)kTileSlots) a.slots[tp * kTileSlots + at] = kk;
      }
      in += (uint32_t)__popcll(m);
    };
    tile_rows(tg.piece, sv.x, held, q, tile_at(a, p.n, t),
              [&](uint2 ent, bool ok) __attribute__((always_inline)) {
                const uint32_t kk = ent.y & kKeyMask;
                up += ok && kk > khi ? 1u : 0u;
                const bool mid = ok && kk - klo <= width;
                if (__ballot(mid) != 0ull) middle(kk, mid);
              },
              [&](uint4 v, uint32_t, uint32_t there) __attribute__((always_inline)) {
                const uint32_t kk[4] = {v.x & kKeyMask, v.y & kKeyMask, v.z & kKeyMask, v.w & kKeyMask};
                bool mid[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                  const bool ok = (there >> e) & 1u;
                  up += ok && kk[e] > khi ? 1u : 0u;
                  mid[e] = ok && kk[e] - klo <= width;
                }
                if (__ballot(mid[0] || mid[1] || mid[2] || mid[3]) == 0ull) return;
#pragma unroll
                for (int e = 0; e < 4; ++e) middle(kk[e], mid[e]);
              });
    if (LEVEL == 1) {
      up = (uint32_t)wave_allsum_u64(up);
      if (lane < (held != kTileOverflow ? (uint32_t)kTileWaves : 1u)) {  // (the other parts of a tile with a piece are empty)
        a.above[tp + lane] = lane == 0u ? up : 0u;
        a.among[tp + lane] = lane == 0u ? in : 0u;
      }
    }
  });
  __syncthreads();
  tile_flush<T>(lh, LEVEL == 1 ? sv.hist1 : sv.hist2);
}

// The threshold itself: pk.lo is the key, pk.need of the pk.cand entries that have it are kept.
template <int T>
__device__ __forceinline__ TilePick tile_threshold(const SegView& sv, uint32_t* part, uint32_t* res, uint32_t* __restrict__ err,
                                                   uint32_t* top = nullptr) {
  TilePick pk = tile_first<T>(sv, part, res, err);
  if (top != nullptr) *top = pk.lo + ((1u << pk.bits) - 1u);
  tile_narrow<T>(pk, sv.hist1, tile_rest(pk.bits), part, res, err);
  if (pk.bits != 0u) {  // (the same in every thread; only the first 128 counts of hist2 are the digit's)
    TileBins<T> tb;
#pragma unroll
    for (int j = 0; j < TileBins<T>::BPT; ++j) {
      const int b = TileBins<T>::BPT * (int)threadIdx.x + j;
      tb.h[j] = b < 128 ? sv.hist2[b] : 0u;
    }
    tile_take(tb, pk, 0u, part, res, err);
  }
  return pk;
}

// ---------------------------------------------------------------------------
// k_tiles_count : per tile the entries above the threshold and at it; only tiles with keys in the bin have anything to look
// at, and most of those all of them in their few slots.
// ---------------------------------------------------------------------------
template <bool APART>
__global__ void __launch_bounds__(64 * kTileWaves)
k_tiles_count(SelParams p, TileArgs a) {
  constexpr int T = 64 * kTileWaves;
  __shared__ uint32_t part[T];
  __shared__ uint32_t res[4];
  __shared__ unsigned long long kept_sh[kTileWaves];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t lane = lane_id();
  if (*p.err != 0u) return;
  const TileGroup<APART> tg(p, a, wave);
  const SegView sv = seg_view(p, tg.seg);
  if (threadIdx.x < kTileWaves) kept_sh[threadIdx.x] = 0ull;
  uint32_t top;  // the last key of the bin
  const TilePick pk = tile_threshold<T>(sv, part, res, p.err, &top);
  const uint32_t width = top - pk.lo;
  tg.each(wave, [&](int i, uint32_t held, int q) __attribute__((always_inline)) {
    const int64_t t = tg.begin + tg.tile(i), tp = t * kTileWaves + q;
    const uint32_t in = __builtin_amdgcn_readfirstlane(a.among[tp]);
    uint64_t kept = (uint64_t)a.above[tp] << 32;
    if (in != 0u) {
      uint32_t up = 0u, eq = 0u;  // a lane's own
      auto one = [&](uint32_t kk, bool ok) __attribute__((always_inline)) {
        up += ok && kk - pk.lo - 1u < width ? 1u : 0u;
        eq += ok && kk == pk.lo ? 1u : 0u;
      };
      if (in <= (uint32_t)kTileSlots) {
        const bool ok = lane < in;
        one(a.slots[tp * kTileSlots + (ok ? lane : 0u)], ok);
      } else {
        tile_rows(tg.piece, sv.x, held, q, tile_at(a, p.n, t), [&](uint2 ent, bool ok) { one(ent.y & kKeyMask, ok); },
                  [&](uint4 v, uint32_t, uint32_t there) __attribute__((always_inline)) {
                    one(v.x & kKeyMask, (there & 1u) != 0u);
                    one(v.y & kKeyMask, (there & 2u) != 0u);
                    one(v.z & kKeyMask, (there & 4u) != 0u);
                    one(v.w & kKeyMask, (there & 8u) != 0u);
                  });
      }
      kept += wave_allsum_u64(((uint64_t)up << 32) | eq);
      if (lane == 0u) {
        a.above[tp] = (uint32_t)(kept >> 32);
        a.among[tp] = (uint32_t)kept;
      }
    }
    if (lane == 0u) atomicAdd(&kept_sh[i], (unsigned long long)kept);
  });
  __syncthreads();
  if (threadIdx.x < kTileWaves && tg.tile((int)threadIdx.x) < tg.ntiles)
    a.kept[tg.begin + tg.tile((int)threadIdx.x)] = kept_sh[threadIdx.x];
  if (threadIdx.x == 0) {
    uint64_t sum = 0ull;
#pragma unroll
    for (int i = 0; i < kTileWaves; ++i) sum += kept_sh[i];
    a.kept[a.ntiles + (int)blockIdx.x] = sum;
  }
}

// ---------------------------------------------------------------------------
// k_tiles_out : the kept entries, in order: what the tiles in front of each of a block's keep is added up first (by block,
// or where the block's tiles lie apart by tile, a wave for each).  With zero_vec the kept entries become +0.0 there, those
// that were at the marking already and are not kept get their values back.
// ---------------------------------------------------------------------------
template <bool APART>
__global__ void __launch_bounds__(64 * kTileWaves)
k_tiles_out(SelParams p, TileArgs a) {
  constexpr int T = 64 * kTileWaves;
  __shared__ uint32_t part[T];
  __shared__ uint32_t res[4];
  __shared__ uint64_t wsum[kTileWaves];
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t lane = lane_id();
  if (*p.err != 0u) return;
  const TileGroup<APART> tg(p, a, wave);
  const SegView sv = seg_view(p, tg.seg);
  const TilePick pk = tile_threshold<T>(sv, part, res, p.err);
  // above the threshold << 32 | at it
  const uint64_t* __restrict__ front = a.kept + (APART ? tg.begin : (int64_t)a.ntiles + sv.d.group_begin);
  const int count = APART ? (tg.tile(wave) < tg.ntiles ? tg.tile(wave) : 0) : tg.number;
  const int step = APART ? 64 : T;
  uint64_t sum = 0ull;
  for (int i = APART ? (int)lane : tid; i < count; i += 4 * step) {  // four in flight
    uint64_t v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = front[i + q * step < count ? i + q * step : i];
#pragma unroll
    for (int q = 0; q < 4; ++q) sum += i + q * step < count ? v[q] : 0ull;
  }
  sum = wave_allsum_u64(sum);
  if (lane == 0u) wsum[wave] = sum;
  __syncthreads();
  const uint32_t key = pk.lo, quota = pk.need, k = sv.d.k;
  const uint32_t zero = p.zero_base[(size_t)tg.seg * kSegWords + kTileInfo + kTileZero];
  float* const zv = p.zero_vec;
  uint32_t nA = 0u, nB = 0u;
  auto place = [&](uint32_t up, uint32_t eq) { return up + (eq < quota ? eq : quota); };
  auto keep = [&](uint32_t m, uint32_t j, uint32_t raw) {
    if (m >= k) return;
    sv.idx_out[m] = (int32_t)j;
    if (sv.vals_row) sv.vals_row[m] = __uint_as_float(raw);
  };
  tg.each(wave, [&](int i, uint32_t held, int q) __attribute__((always_inline)) {
    const int ts = tg.tile(i);
    const int64_t t = tg.begin + ts;
    uint64_t ahead = 0ull;
    if (APART) {
      ahead = wsum[i];
    } else {
#pragma unroll
      for (int w = 0; w < kTileWaves; ++w) ahead += wsum[w];
      for (int w = 0; w < i; ++w) ahead += a.kept[t - i + w];
    }
    for (int w = 0; w < q; ++w) ahead += ((uint64_t)a.above[t * kTileWaves + w] << 32) | a.among[t * kTileWaves + w];
    nA = (uint32_t)(ahead >> 32);
    nB = (uint32_t)ahead;
    if (a.tile_start != nullptr && lane == 0u && q == 0) {
      static_assert(kPassTile == 2 * kMarkTile, "two tiles");
      if ((t & 1) == 0) a.tile_start[t >> 1] = (int32_t)sv.d.koff + (int32_t)place(nA, nB);
      if (ts == tg.ntiles - 1) a.tile_start[(t + 2) >> 1] = (int32_t)sv.d.koff + (int32_t)k;
    }
    tile_rows(tg.piece, sv.x, held, q, tile_at(a, p.n, t),
              [&](uint2 ent, bool ok) __attribute__((always_inline)) {
                const uint32_t kk = ent.y & kKeyMask;
                const bool up = ok && kk > key, eq = ok && kk == key;
                const uint64_t mu = __ballot(up), me = __ballot(eq);
                const uint32_t before = nB + popc_lt(me);
                const bool kept = up || (eq && before < quota);
                if (kept) keep(place(nA + popc_lt(mu), before), ent.x, ent.y);
                if (zv != nullptr && ok && (int64_t)ent.x < p.n) {
                  if (kept && kk < zero) zv[ent.x] = 0.0f;
                  if (!kept && kk >= zero) zv[ent.x] = __uint_as_float(ent.y);
                }
                nA += (uint32_t)__popcll(mu);
                nB += (uint32_t)__popcll(me);
              },
              [&](uint4 v, uint32_t j, uint32_t there) __attribute__((always_inline)) {
                const uint32_t raw[4] = {v.x, v.y, v.z, v.w};
                bool up[4], eq[4];
                uint64_t mu[4], me[4];
  #pragma unroll
                for (int e = 0; e < 4; ++e) {
                  const uint32_t kk = raw[e] & kKeyMask;
                  up[e] = ((there >> e) & 1u) && kk > key;
                  eq[e] = ((there >> e) & 1u) && kk == key;
                  mu[e] = __ballot(up[e]);
                  me[e] = __ballot(eq[e]);
                }
                if ((mu[0] | mu[1] | mu[2] | mu[3] | me[0] | me[1] | me[2] | me[3]) == 0ull) return;
                uint32_t bu = nA, be = nB;
  #pragma unroll
                for (int e = 0; e < 4; ++e) {
                  bu += popc_lt(mu[e]);
                  nA += (uint32_t)__popcll(mu[e]);
                }
                if ((me[0] | me[1] | me[2] | me[3]) != 0ull) {
  #pragma unroll
                  for (int e = 0; e < 4; ++e) {
                    be += popc_lt(me[e]);
                    nB += (uint32_t)__popcll(me[e]);
                  }
                }
  #pragma unroll
                for (int e = 0; e < 4; ++e) {
                  if (up[e] || (eq[e] && be < quota)) {
                    keep(place(bu, be), j + (uint32_t)e, raw[e]);
                    if (zv != nullptr) zv[j + (uint32_t)e] = 0.0f;
                  }
                  bu += up[e] ? 1u : 0u;
                  be += eq[e] ? 1u : 0u;
                }
              });
  });
}

// ---------------------------------------------------------------------------
// k_tile_starts : tile_start[t] = number of kept indices below t * kPassTile, for
// t = 0 .. ntiles (so tile_start[ntiles] = k), from the ascending index list.
// One thread per index: idx[p] owns the entries of the tiles that begin between
// idx[p-1] and idx[p], the last index also the rest; the 64 lanes of a wave fill
// each owner's entries together, so a long run of empty tiles costs its length / 64.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
k_tile_starts(const int32_t* __restrict__ idx, int64_t k, int32_t ntiles, int32_t* __restrict__ tile_start) {
  const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int lane = threadIdx.x & 63;
  int32_t t0 = 1, t1 = 0, t_last = -1;  // [t0, t1] = entries this index owns (empty by default)
  if (p < k) {
    const int64_t i = (int64_t)idx[p];
    const int64_t prev = p > 0 ? (int64_t)idx[p - 1] : -1;
    if (i >= 0 && i >= prev) {  // otherwise not an ascending index list: k_pass_rest reports what is left unset
      const int64_t t = i / kPassTile;
      t1 = (int32_t)(t < ntiles ? t : ntiles);
      t0 = prev < 0 ? 0 : (int32_t)(prev / kPassTile) + 1;
      if (p == k - 1) t_last = t1;
    }
  }
  uint64_t todo = __ballot(t0 <= t1);
  while (todo != 0ull) {
    const int src = __ffsll((unsigned long long)todo) - 1;
    todo &= todo - 1;
    const int32_t a = __shfl(t0, src, 64), b = __shfl(t1, src, 64);
    const int32_t v = (int32_t)(p - lane + src);
    for (int32_t t = a + lane; t <= b; t += 64) tile_start[t] = v;
  }
  const uint64_t fin = __ballot(t_last >= 0);
  if (fin != 0ull) {
    const int src = __ffsll((unsigned long long)fin) - 1;
    const int32_t a = __shfl(t_last, src, 64) + 1;
    for (int32_t t = a + lane; t <= ntiles; t += 64) tile_start[t] = (int32_t)k;
  }
}

// ---------------------------------------------------------------------------
// k_tile_starts_search : the same table when there are many more kept indices than
// tiles: one thread per entry t looks up the first position whose index is not
// below t * kPassTile (binary search in the ascending list; the upper levels of the
// search are shared by all threads and stay in the cache).  A list that does not
// ascend gives bounds that k_pass_rest / k_update_tiles reject or clip.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
k_tile_starts_search(const int32_t* __restrict__ idx, int64_t k, int32_t ntiles, int32_t* __restrict__ tile_start) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t > ntiles) return;
  const int64_t target = t * kPassTile;
  int64_t lo = 0, hi = k;  // the answer lies in [lo, hi]
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if ((int64_t)idx[mid] < target) lo = mid + 1; else hi = mid;
  }
  tile_start[t] = (int32_t)lo;
}

// ---------------------------------------------------------------------------
// k_pass_rest : for every worker except the leader, in one streaming pass:
//   acc = g + residual; at the kept indices vals[w][m] = acc and the residual
//   becomes +0.0, elsewhere the residual becomes acc.
// Used when the leader is known before the step starts (its own pass and the
// selection have already run, so idx is final and k_tile_starts has run).
// grid = (gx, W-1), block = T; block (b, y) works on worker (leader + 1 + y) mod W
// and takes the tiles b, b + gx, ... of T U float4 groups (see k_pass_mark).  Per
// tile it marks the kept positions, idx[tile_start[t] .. tile_start[t+1]), in an
// LDS slot table while the tile's loads are in flight.
// ---------------------------------------------------------------------------
template <bool NT, int GT, int T, int U>
__global__ void __launch_bounds__(T)
k_pass_rest(PtrTable g, PtrTable res, int w_count, int leader, int64_t n, const int32_t* __restrict__ idx, int64_t k,
            float* __restrict__ vals, const int32_t* __restrict__ tile_start, uint32_t* __restrict__ err) {
  constexpr int TILE = T * 4 * U;  // elements per tile: T threads x U float4
  static_assert(TILE == kPassTile, "tile_start is laid out for this tile");
  static_assert(TILE <= 32768, "slot entries are 16-bit offsets from the tile's first index");
  __shared__ __attribute__((aligned(16))) int16_t slot[TILE];
  const int tid = threadIdx.x;
  const int w = (int)(((unsigned)leader + 1u + blockIdx.y) % (unsigned)w_count);
  const float* __restrict__ gp = g.p[w];
  float* __restrict__ rp = res.p[w];
  float* __restrict__ vrow = vals + (size_t)w * (size_t)k;
  uint2* s2 = reinterpret_cast<uint2*>(slot);  // four 16-bit slots: one float4 group

  const int64_t q_end = n >> 2;  // whole float4 groups end here
  const int64_t ntiles = q_end > 0 ? (n + TILE - 1) / TILE : 0;  // fewer than four elements: only the scalar tail
  // The counter that loads are waited on counts them in issue order, so whatever is needed early
  // is issued early: the bounds of the NEXT tile's indices one tile ahead, this tile's indices
  // before its big loads; the slot table is then filled while those are in flight.
  int64_t ti = blockIdx.x;
  int32_t m0 = 0, m1 = 0;
  if (ti < ntiles) {
    m0 = tile_start[ti];
    m1 = tile_start[ti + 1];
  }
  for (; ti < ntiles; ti += gridDim.x) {
    const int64_t ti_next = ti + gridDim.x;
    int32_t n0 = 0, n1 = 0;
    if (ti_next < ntiles) {
      n0 = tile_start[ti_next];
      n1 = tile_start[ti_next + 1];
    }
    int64_t m_base = (int64_t)m0, m_end = (int64_t)m1;
    if (m_base < 0 || m_end > k || m_end < m_base || m_end - m_base > TILE) {  // idx was not ascending
      if (tid == 0) atomicOr(err, kErrIndex);
      m_end = m_base = 0;
    }
    const int64_t lo = ti * TILE;
    // (no branch around the load: beyond the tile's indices it re-reads the last index, unused)
    const int64_t p0 = m_base + tid;
    const int32_t i0 = idx[p0 < m_end ? p0 : k - 1];
    const int64_t q0 = (lo >> 2) + tid;
    const bool full = lo + TILE <= 4 * q_end;
    v4f a[U], b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      // groups behind the vector re-read its last group (unused): no branch between or around the
      // loads, or the compiler would wait for all of them before the first use of an index
      const int64_t q = q0 + u * T;
      const int64_t ql = (full || q < q_end) ? q : q_end - 1;
      a[u] = load4g<NT, GT>(gp, 4 * ql);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {  // (one array after the other: see k_pass_mark)
      const int64_t q = q0 + u * T;
      const int64_t ql = (full || q < q_end) ? q : q_end - 1;
      b[u] = load4<NT>(rp + 4 * ql);
    }
    // slot[j] = (position in idx) - m_base for a kept element j of this tile, else -1
#pragma unroll
    for (int u = 0; u < U; ++u) s2[tid + u * T] = make_uint2(0xffffffffu, 0xffffffffu);
    __syncthreads();
    {
      const int64_t i = (int64_t)i0 - lo;
      if (p0 < m_end && i >= 0 && i < TILE) slot[i] = (int16_t)tid;
    }
    for (int64_t p = p0 + T; p < m_end; p += T) {  // dense tiles only (more than T kept of 32 T elements)
      const int64_t i = (int64_t)idx[p] - lo;
      if (i >= 0 && i < TILE) slot[i] = (int16_t)(p - m_base);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t q = q0 + u * T;
      if (full || q < q_end) {
        const uint2 sl = s2[tid + u * T];
        v4f v;
        v.x = a[u].x + b[u].x;
        v.y = a[u].y + b[u].y;
        v.z = a[u].z + b[u].z;
        v.w = a[u].w + b[u].w;
        if ((sl.x & sl.y) != 0xffffffffu) {  // some element of this group is kept
          const int s0 = (int16_t)(sl.x & 0xffffu), s1 = (int16_t)(sl.x >> 16);
          const int s2v = (int16_t)(sl.y & 0xffffu), s3 = (int16_t)(sl.y >> 16);
          if (s0 >= 0) { vrow[m_base + s0] = v.x; v.x = 0.0f; }
          if (s1 >= 0) { vrow[m_base + s1] = v.y; v.y = 0.0f; }
          if (s2v >= 0) { vrow[m_base + s2v] = v.z; v.z = 0.0f; }
          if (s3 >= 0) { vrow[m_base + s3] = v.w; v.w = 0.0f; }
        }
        store4<NT>(rp + 4 * q, v);
      }
    }
    __syncthreads();  // the slot table is rebuilt for the next tile
    m0 = n0;
    m1 = n1;
  }
  // scalar tail of the vector (n not a multiple of 4): the first block
  if (blockIdx.x == 0) {
    const int64_t j = (n >> 2) * 4 + tid;
    if (j < n) {
      float v = load1g<GT>(gp, j) + rp[j];
      int64_t lo = 0, hi = k;  // binary search for j among the indices
      while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t)idx[mid] < j) lo = mid + 1; else hi = mid;
      }
      if (lo < k && (int64_t)idx[lo] == j) {
        vrow[lo] = v;
        v = 0.0f;
      }
      rp[j] = v;
    }
  }
}

// ---------------------------------------------------------------------------
// k_sum_rows : sum[m] = ((vals[0][m] + vals[1][m]) + ...) + vals[W-1][m], float32,
// in that order.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
k_sum_rows(const float* __restrict__ vals, int w_count, int64_t k, float* __restrict__ sum) {
  const int64_t m0 = (int64_t)blockIdx.x * 1024 + threadIdx.x;  // this thread: m0, m0+256, m0+512, m0+768
  float s[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  for (int w0 = 0; w0 < w_count; w0 += 4) {  // sixteen independent loads in flight, then the ordered adds
    float v[4][4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (w0 + j < w_count && m0 + e * 256 < k) v[j][e] = vals[(size_t)(w0 + j) * (size_t)k + (size_t)(m0 + e * 256)];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (w0 + j < w_count && m0 + e * 256 < k) s[e] = (w0 + j == 0) ? v[j][e] : (s[e] + v[j][e]);
  }
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (m0 + e * 256 < k) sum[m0 + e * 256] = s[e];
}

// ---------------------------------------------------------------------------
// k_gather : one thread per kept index m.  vals[w][m] = x_w[idx[m]], sum[m] is
// the float32 sum over w = 0, 1, ..., W-1 in that order; with ZERO the
// position is then overwritten by +0.0 in every worker.
// ---------------------------------------------------------------------------
template <bool ZERO>
__global__ void __launch_bounds__(256)
k_gather(PtrTable tab, int w_count, int64_t n, const int32_t* __restrict__ idx, int64_t k,
         float* __restrict__ vals, float* __restrict__ sum, uint32_t* __restrict__ err) {
  const int64_t m = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (m >= k) return;
  const int64_t i = (int64_t)idx[m];
  if (i < 0 || i >= n) {  // never touch memory through an index outside the vector
    atomicOr(err, kErrIndex);
    return;
  }
  float s = 0.0f;
  for (int w0 = 0; w0 < w_count; w0 += 8) {  // eight independent loads in flight, then the ordered adds
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (w0 + j < w_count) v[j] = tab.p[w0 + j][i];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (w0 + j < w_count) {
        if (vals) vals[(size_t)(w0 + j) * (size_t)k + (size_t)m] = v[j];
        s = (w0 + j == 0) ? v[j] : (s + v[j]);
        if (ZERO) tab.p[w0 + j][i] = 0.0f;
      }
    }
  }
  if (sum) sum[m] = s;
}

// ---------------------------------------------------------------------------
// k_zero_at : +0.0 at the kept indices of every worker, from the last ones on: a gather that went before has left the lines
// of those in the last-level cache (2 x 2.8 M of 138 M, the whole exchange 440 us forwards, 435 backwards).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
k_zero_at(PtrTable tab, int w_count, int64_t n, const int32_t* __restrict__ idx, int64_t k,
          uint32_t* __restrict__ err) {
  const int64_t m = (int64_t)(gridDim.x - 1u - blockIdx.x) * 256 + threadIdx.x;
  if (m >= k) return;
  const int64_t i = (int64_t)idx[m];
  if (i < 0 || i >= n) {
    atomicOr(err, kErrIndex);
    return;
  }
  for (int w = 0; w < w_count; ++w) tab.p[w][i] = 0.0f;
}

// ---------------------------------------------------------------------------
// k_update_fill : update = zeros(N) with update[idx[m]] = sum[m], every output
// element written exactly once.  Block b owns a contiguous run of 8192-element
// chunks; it locates its first index with a 256-way search, then per chunk
// builds the chunk in LDS (BATCH x 256 index/sum pairs per round, fetched ahead
// of the buffer clear) and streams it out.
// ---------------------------------------------------------------------------
constexpr int kFillChunk = 8192;

// What a thread holds of the (index, sum) pairs ahead of the chunk being built.
template <int BATCH>
struct FillAhead {
  int64_t ib[BATCH];
  float sb[BATCH];
};

constexpr int64_t kFillNone = INT64_MAX;  // no index: beyond every chunk

template <int BATCH>
__device__ __forceinline__ void fill_fetch(FillAhead<BATCH>& a, const int32_t* __restrict__ idx,
                                           const float* __restrict__ sum, int64_t k, int64_t from) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int j = 0; j < BATCH; ++j) {
    // (no branch around the loads: behind the list they re-read its last entry, unused)
    const int64_t p = from + tid + j * 256;
    const int64_t pc = p < k ? p : k - 1;
    const int32_t iv = idx[pc];
    const float sv = sum[pc];
    a.ib[j] = p < k ? (int64_t)iv : kFillNone;
    a.sb[j] = sv;
  }
}

// Builds and streams out the chunks [c_begin, c_end) of the update; m = number of indices below
// the first of them, whose first pairs `a` already holds.  The pairs a chunk starts with are
// fetched one chunk ahead, before the previous chunk is streamed out, so that their latency is
// not part of the chunk's own chain; behind the last chunk the fetch goes to m_after (the start
// of the block's next run) if that is not negative.  All 256 threads call it.
template <int BATCH>
__device__ __forceinline__ void fill_run(FillAhead<BATCH>& a, float* __restrict__ buf, float* __restrict__ update,
                                         int64_t n, const int32_t* __restrict__ idx, const float* __restrict__ sum,
                                         int64_t k, int64_t c_begin, int64_t c_end, int64_t m, int64_t m_after) {
  constexpr int kGroups = kFillChunk / 4 / 256;  // float4 groups per thread and chunk
  const int tid = threadIdx.x;
  for (int64_t c = c_begin; c < c_end; ++c) {
    const int64_t lo = c * kFillChunk;
    const int64_t hi = (lo + kFillChunk < n) ? lo + kFillChunk : n;
    const int64_t len = hi - lo;
    const int64_t len4 = len >> 2;
    float4* b4 = reinterpret_cast<float4*>(buf);
    for (int i = tid; i < kFillChunk / 4; i += 256) b4[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    __syncthreads();
    while (true) {
      int cnt = 0;
#pragma unroll
      for (int j = 0; j < BATCH; ++j) {
        const bool in = a.ib[j] < hi;
        if (in && a.ib[j] >= lo) {  // ib >= lo always holds for ascending idx
          const int64_t off = a.ib[j] - lo;
          buf[off] = a.sb[j];
        }
        cnt += __syncthreads_count(in);
      }
      m += cnt;
      const bool chunk_done = cnt < BATCH * 256;
      // the next chunk's first pairs, or the rest of this chunk's
      fill_fetch<BATCH>(a, idx, sum, k, (chunk_done && c == c_end - 1 && m_after >= 0) ? m_after : m);
      if (chunk_done) break;
    }
    // (the count barrier above also orders the LDS writes before the reads)
    float* __restrict__ up = update + lo;
#pragma unroll
    for (int j = 0; j < kGroups; ++j) {
      const int64_t i = tid + j * 256;
      if (i < len4) {
        // (non-temporal: with ordinary stores the time of this fill depended on what earlier
        // kernels had left in the caches, 115 to 150 us on 138 M elements; so it is 115 throughout)
        const float4 t4 = b4[i];
        const v4f tv = {t4.x, t4.y, t4.z, t4.w};
        store4<true>(up + 4 * i, tv);
      }
    }
    for (int64_t i = len4 * 4 + tid; i < len; i += 256) up[i] = buf[i];  // ragged end of the vector
    __syncthreads();
  }
}

template <int BATCH>
__global__ void __launch_bounds__(256)
k_update_fill(float* __restrict__ update, int64_t n, const int32_t* __restrict__ idx,
              const float* __restrict__ sum, int64_t k) {
  __shared__ __attribute__((aligned(16))) float buf[kFillChunk];
  __shared__ int64_t s_lo, s_hi;
  const int tid = threadIdx.x;
  const int64_t nchunk = (n + kFillChunk - 1) / kFillChunk;
  const int64_t c_begin = nchunk * (int64_t)blockIdx.x / (int64_t)gridDim.x;
  const int64_t c_end = nchunk * ((int64_t)blockIdx.x + 1) / (int64_t)gridDim.x;
  if (c_begin >= c_end) return;

  // m = number of indices below the first element of this block's run
  const int64_t target = c_begin * kFillChunk;
  if (tid == 0) {
    s_lo = 0;
    s_hi = k;
  }
  __syncthreads();
  while (true) {
    const int64_t lo = s_lo, hi = s_hi;  // answer lies in [lo, hi]
    const int64_t span = hi - lo;
    if (span <= 0) break;
    const int64_t stepw = (span + 255) / 256;
    const int64_t p = lo + (int64_t)tid * stepw;  // probe positions lo, lo+stepw, ...
    const bool below = (p < hi) && ((int64_t)idx[p] < target);
    const int cnt = __syncthreads_count(below);
    // probes 0..cnt-1 are below the target: the answer is in (lo+(cnt-1)*stepw, lo+cnt*stepw]
    if (tid == 0) {
      if (cnt == 0) {
        s_hi = lo;
      } else {
        const int64_t nlo = lo + (int64_t)(cnt - 1) * stepw + 1;
        int64_t nhi = lo + (int64_t)cnt * stepw;
        if (nhi > hi) nhi = hi;
        s_lo = nlo;
        s_hi = nhi;
      }
    }
    __syncthreads();
  }
  const int64_t m = s_lo;
  FillAhead<BATCH> a;
  fill_fetch<BATCH>(a, idx, sum, k, m);
  fill_run<BATCH>(a, buf, update, n, idx, sum, k, c_begin, c_end, m, -1);
}

// The same with the blocks striding over the tiles of the streaming passes (kPassTile elements, four
// chunks), whose first indices k_tile_starts has left in tile_start: no search, and at any time the
// blocks in flight write one contiguous window of the update.
template <int BATCH>
__global__ void __launch_bounds__(256)
k_update_fill_tiled(float* __restrict__ update, int64_t n, const int32_t* __restrict__ idx,
                    const float* __restrict__ sum, int64_t k, const int32_t* __restrict__ tile_start) {
  __shared__ __attribute__((aligned(16))) float buf[kFillChunk];
  constexpr int64_t kPer = kPassTile / kFillChunk;  // chunks per tile
  const int64_t nchunk = (n + kFillChunk - 1) / kFillChunk;
  const int64_t ntiles = (n + kPassTile - 1) / kPassTile;
  // (a start outside [0, k] can only come from an index list that was not ascending)
  auto start_of = [&](int64_t t) {
    const int64_t v = (int64_t)tile_start[t];
    return v < 0 ? (int64_t)0 : (v > k ? k : v);
  };
  int64_t ti = blockIdx.x;
  if (ti >= ntiles) return;
  int64_t m = start_of(ti);
  FillAhead<BATCH> a;
  fill_fetch<BATCH>(a, idx, sum, k, m);
  for (; ti < ntiles; ti += gridDim.x) {
    const int64_t tn = ti + gridDim.x;
    const int64_t m_next = tn < ntiles ? start_of(tn) : k;
    const int64_t c_begin = ti * kPer;
    const int64_t c_end = c_begin + kPer < nchunk ? c_begin + kPer : nchunk;
    fill_run<BATCH>(a, buf, update, n, idx, sum, k, c_begin, c_end, m, m_next);
    m = m_next;
  }
}

// ---------------------------------------------------------------------------
// k_update_tiles : the same dense update for long vectors: zeros streamed out tile
// by tile (kPassTile elements, blocks striding over the tiles as in k_pass_mark), and
// behind a tile's zeros the same block stores sum[m] at the tile's kept indices,
// idx[tile_start[t] .. tile_start[t+1]) (k_tile_starts has run).  The barrier between
// the two orders them for the block's stores to one address; the lines are still in
// the cache when the second store arrives, so memory sees each line once.
// NTZ: the zeros go out as non-temporal stores (measured per step: better on 138 M
// elements, 1.335 against 1.354 ms, because the kernels that follow find less of this
// vector in the caches; worse on 1e9, 654 against 626 us for the kernel itself).
// ---------------------------------------------------------------------------
template <int T, int U, bool NTZ>
__global__ void __launch_bounds__(T)
k_update_tiles(float* __restrict__ update, int64_t n, const int32_t* __restrict__ idx, const float* __restrict__ sum,
               int64_t k, const int32_t* __restrict__ tile_start, uint32_t* __restrict__ err) {
  constexpr int TILE = T * 4 * U;
  static_assert(TILE == kPassTile, "tile_start is laid out for this tile");
  const int tid = threadIdx.x;
  const int64_t q_end = n >> 2;  // whole float4 groups
  const int64_t ntiles = (n + TILE - 1) / TILE;
  const v4f zero = {0.f, 0.f, 0.f, 0.f};
  int64_t ti = blockIdx.x;
  int32_t m0 = 0, m1 = 0;
  if (ti < ntiles) {
    m0 = tile_start[ti];
    m1 = tile_start[ti + 1];
  }
  for (; ti < ntiles; ti += gridDim.x) {
    const int64_t ti_next = ti + gridDim.x;
    int32_t n0 = 0, n1 = 0;
    if (ti_next < ntiles) {  // the next tile's bounds, one tile ahead
      n0 = tile_start[ti_next];
      n1 = tile_start[ti_next + 1];
    }
    int64_t m_base = (int64_t)m0, m_end = (int64_t)m1;
    if (m_base < 0 || m_end > k || m_end < m_base || m_end - m_base > TILE) {  // idx was not ascending
      if (tid == 0) atomicOr(err, kErrIndex);
      m_end = m_base = 0;
    }
    const int64_t lo = ti * TILE;
    // this tile's first T (index, sum) pairs, fetched while the zeros go out
    // (no branch around the loads: behind the tile's pairs they re-read the last pair, unused)
    const int64_t p0 = m_base + tid;
    const int64_t pc = p0 < m_end ? p0 : k - 1;
    const int32_t i0 = idx[pc];
    const float s0 = sum[pc];
    const int64_t q0 = (lo >> 2) + tid;
    if (lo + TILE <= 4 * q_end) {
#pragma unroll
      for (int u = 0; u < U; ++u) store4<NTZ>(update + 4 * (q0 + u * T), zero);
    } else {  // the last tile: whole groups, then the ragged end
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (q0 + u * T < q_end) store4<NTZ>(update + 4 * (q0 + u * T), zero);
      const int64_t j = 4 * q_end + tid;
      if (j < n) update[j] = 0.0f;
    }
    __syncthreads();  // the block's zeros are ordered before its values
    if (p0 < m_end) {
      const int64_t i = (int64_t)i0 - lo;
      if (i >= 0 && i < TILE && lo + i < n) update[lo + i] = s0;
    }
    for (int64_t p = p0 + T; p < m_end; p += T) {  // dense tiles only
      const int64_t i = (int64_t)idx[p] - lo;
      if (i >= 0 && i < TILE && lo + i < n) update[lo + i] = sum[p];
    }
    m0 = n0;
    m1 = n1;
  }
}

// ---------------------------------------------------------------------------
// k_sum_update : the end of a step whose leader was known up front, behind the
// other workers' pass: sum[m] = ((vals[0][m] + vals[1][m]) + ...) + vals[W-1][m] in
// float32, in that order, and the dense update, zeros with sum[m] at idx[m], every
// element written once.  Blocks stride over the tiles as in k_pass_rest and mark a
// tile's kept positions, idx[tile_start[t] .. tile_start[t+1]), in the same 16-bit
// slot table; the thread that owns a kept position adds up the rows' entries and
// stores the sum on its way through the tile's float4 groups.
// ---------------------------------------------------------------------------
template <int T, int U>
__global__ void __launch_bounds__(T)
k_sum_update(const float* __restrict__ vals, int w_count, int64_t n, const int32_t* __restrict__ idx, int64_t k,
             const int32_t* __restrict__ tile_start, float* __restrict__ sum_out, float* __restrict__ update,
             uint32_t* __restrict__ err) {
  constexpr int TILE = T * 4 * U;
  static_assert(TILE == kPassTile, "tile_start is laid out for this tile");
  static_assert(TILE <= 32768, "slot entries are 16-bit offsets from the tile's first index");
  __shared__ __attribute__((aligned(16))) int16_t slot[TILE];
  const int tid = threadIdx.x;
  uint2* s2 = reinterpret_cast<uint2*>(slot);  // four 16-bit slots: one float4 group
  const int64_t q_end = n >> 2;  // whole float4 groups end here
  const int64_t ntiles = q_end > 0 ? (n + TILE - 1) / TILE : 0;

  // sum of the rows' entries at position m, in worker order
  auto ordered_sum = [&](int64_t m) {
    float sacc = vals[m];
    for (int w = 1; w < w_count; ++w) sacc = sacc + vals[(size_t)w * (size_t)k + (size_t)m];
    return sacc;
  };

  int64_t ti = blockIdx.x;
  int32_t m0 = 0, m1 = 0;
  if (ti < ntiles) {
    m0 = tile_start[ti];
    m1 = tile_start[ti + 1];
  }
  for (; ti < ntiles; ti += gridDim.x) {
    const int64_t ti_next = ti + gridDim.x;
    int32_t n0 = 0, n1 = 0;
    if (ti_next < ntiles) {  // the next tile's bounds, one tile ahead
      n0 = tile_start[ti_next];
      n1 = tile_start[ti_next + 1];
    }
    int64_t m_base = (int64_t)m0, m_end = (int64_t)m1;
    if (m_base < 0 || m_end > k || m_end < m_base || m_end - m_base > TILE) {  // idx was not ascending
      if (tid == 0) atomicOr(err, kErrIndex);
      m_end = m_base = 0;
    }
    const int64_t lo = ti * TILE;
    const int64_t p0 = m_base + tid;
    const int32_t i0 = idx[p0 < m_end ? p0 : k - 1];
    const int64_t q0 = (lo >> 2) + tid;
    const bool full = lo + TILE <= 4 * q_end;
#pragma unroll
    for (int u = 0; u < U; ++u) s2[tid + u * T] = make_uint2(0xffffffffu, 0xffffffffu);
    __syncthreads();
    {
      const int64_t i = (int64_t)i0 - lo;
      if (p0 < m_end && i >= 0 && i < TILE) slot[i] = (int16_t)tid;
    }
    for (int64_t p = p0 + T; p < m_end; p += T) {  // dense tiles only (more than T kept of 32 T elements)
      const int64_t i = (int64_t)idx[p] - lo;
      if (i >= 0 && i < TILE) slot[i] = (int16_t)(p - m_base);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t q = q0 + u * T;
      if (full || q < q_end) {
        const uint2 sl = s2[tid + u * T];
        v4f z = {0.f, 0.f, 0.f, 0.f};
        if ((sl.x & sl.y) != 0xffffffffu) {  // some element of this group is kept
          const int s0 = (int16_t)(sl.x & 0xffffu), s1 = (int16_t)(sl.x >> 16);
          const int s2v = (int16_t)(sl.y & 0xffffu), s3 = (int16_t)(sl.y >> 16);
          if (s0 >= 0) { z.x = ordered_sum(m_base + s0); sum_out[m_base + s0] = z.x; }
          if (s1 >= 0) { z.y = ordered_sum(m_base + s1); sum_out[m_base + s1] = z.y; }
          if (s2v >= 0) { z.z = ordered_sum(m_base + s2v); sum_out[m_base + s2v] = z.z; }
          if (s3 >= 0) { z.w = ordered_sum(m_base + s3); sum_out[m_base + s3] = z.w; }
        }
        store4<true>(update + 4 * q, z);
      }
    }
    __syncthreads();  // the slot table is rebuilt for the next tile
    m0 = n0;
    m1 = n1;
  }
  // the n mod 4 last elements: the first block
  if (blockIdx.x == 0) {
    const int64_t j = (n >> 2) * 4 + tid;
    if (j < n) {
      int64_t lo = 0, hi = k;  // binary search for j among the indices
      while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t)idx[mid] < j) lo = mid + 1; else hi = mid;
      }
      float upd = 0.0f;
      if (lo < k && (int64_t)idx[lo] == j) {
        upd = ordered_sum(lo);
        sum_out[lo] = upd;
      }
      update[j] = upd;
    }
  }
}

// ---------------------------------------------------------------------------
// k_small_step : a whole flat step on a short vector in one launch.  Bound by latency: three launches, each a chain of
// trips to memory between a start and an end, took 30.6 us on 65537 elements x 2 workers and 55 on 1 M x 4; here the
// blocks wait for each other in between, which takes a microsecond, and the same steps take 17.3 and 27.3.
//   A block has one chunk of 8 T elements, of every worker, and takes it from the gradients to the outputs:
//     acc = g + residual, the counts of the leader's (every worker's, where the leader comes from the data) top digits;
//     all blocks are through with that: threshold digit (every block picks it for itself), the candidates' second digits;
//     all are through: second digit of the threshold, the entries it leaves, per chunk, by their last seven bits;
//     all are through: threshold, how many are kept in front of the chunk, and the outputs of the chunk.
// So a block reads what it wrote itself, except for counts, which go past the XCD's cache (load_through).  With the
// leader known up front the other workers' sums are formed while the block waits.  Many workers of few chunks are shared
// out among further blocks in the first part (small_step's rule); their sums then go past the cache, too.  However many values share the
// threshold's digits, the work is the same (1 M x 2 between 1 and 1.01, one in a hundred kept: 73 us in three launches).
//   Nothing depends on how many blocks run at a time: a block that has looked for the others' first counts for a while
// takes on the chunks that nobody has (a chunk bears the number of the step in which it was taken; a block that comes
// late finds its own taken and leaves), and from then on every chunk belongs to a block that runs.  Everything that is
// counted up is zero again when the step ends, or, of two sets in turn, when the next but one begins.
//   8 T is 4096 up to 2^20 elements and 8192 beyond: at most 256 blocks (us, 2048 / 4096 / 8192: 65537 x 2 21/20/-, 262143
// x 2 25/21/-; variance rule, the best groups of each, 65537 x 8 27/25/30, 262143 x 8 39/32/35, 500009 x 16 77/65/66, 1 M
// x 16 -/79/100).  One copy of a histogram up to 128 chunks, two beyond (one / two / four: 524288 x 4 22.8/24.7/25.0, 1 M
// x 4 28.2/26.6/29.7, 1 M x 8 variance rule 65/54.6/55.6): each more is another 16 KB that every block reads twice, each
// fewer more additions to one place.
// ---------------------------------------------------------------------------
constexpr int kSmallReps = 2;         // copies of a histogram, at most
constexpr int kSmallMaxChunks = 256;  // chunks, at most
constexpr int kSmallMaxUnits = 256;   // chunks x groups of workers, at most
constexpr int kSmallLine = 32;        // words between counters
// SmallScratch::ctr, words: the step's number; chunks that other blocks took on, and blocks that came late, of this
// step; two sets of three waits' counters
constexpr int kCtrStep = 0, kCtrHelped = kSmallLine, kCtrLate = 2 * kSmallLine, kCtrArrive = 3 * kSmallLine,
              kCtrSet = 3 * kMeetWait, kSmallCtr = kCtrArrive + 2 * kCtrSet;
// Few candidates: so many of the vector's, in so many chunks at most (a lane each), are handed on themselves.
constexpr int kSmallFew = 2048, kSmallFewChunks = 64, kSmallRows = kSmallMaxChunks * 128;
// What select_info reports as many candidates (no route depends on it).
__host__ __device__ constexpr uint32_t small_few(int64_t n) { return 10240u + 240u * (uint32_t)((n + kTile - 1) / kTile); }

struct SmallScratch {
  // zero at first
  uint32_t* hist;   // [workers][kSmallReps][kHistBins] top digits
  uint32_t* ctr;    // [kSmallCtr]
  uint32_t* claim;  // [kSmallMaxUnits] the step in which somebody took the chunk of the group, plus one
  uint32_t* dig1;   // [kSmallReps][kHistBins] second digits of the candidates
  uint32_t* dig2;   // [2][kSmallReps][128] last digits of those that are left then
  // written before they are read in every step
  uint32_t* above;  // [kSmallMaxChunks] a chunk's keys above those
  uint32_t* rows;   // [kSmallMaxChunks][128] a chunk's of those: with that last digit or a higher one; or its candidates
};

struct SmallStep {
  PtrTable g, res;
  int64_t n;
  uint32_t k;
  int32_t w_count;
  int32_t leader;  // -1: from the statistics, or in leader_dev
  int32_t nchunks, reps;
  int32_t groups;     // of workers: each has its blocks in the first part (of a known leader: itself, and the others)
  int32_t raw_stats;  // the statistics are the raw gradient's
  uint32_t list_cap;  // (what the state reports of the general selection's list)
  SmallScratch ss;
  double* partials;
  SelState* st;
  uint32_t* err;
  int32_t* leader_dev;
  int32_t* leader_out;
  double* var_out;
  int32_t* idx_out;
  float* vals;
  float* sum_out;
  float* update;
};

// The elements [j0, j0 + 8) of g and of r (those behind the vector unspecified).
template <int GT>
__device__ __forceinline__ void small_fetch(const float* __restrict__ g, const float* __restrict__ r, int64_t n,
                                            int64_t j0, v4f (&a)[2], v4f (&b)[2]) {
  if (j0 + 8 <= n) {
    a[0] = load4g<false, GT>(g, j0);
    a[1] = load4g<false, GT>(g, j0 + 4);
    b[0] = load4<false>(r + j0);
    b[1] = load4<false>(r + j0 + 4);
  } else if (j0 < n) {  // one thread of the vector's (behind its end the last element again, unused)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int64_t j = j0 + e < n ? j0 + e : n - 1;
      a[e >> 2][e & 3] = load1g<GT>(g, j);
      b[e >> 2][e & 3] = r[j];
    }
  }
}

// Adds the occupied bins of the block's histogram to dst and clears it.
template <int T>
__device__ __forceinline__ void small_flush(uint32_t* __restrict__ lh, uint32_t* __restrict__ dst) {
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kHistBins / T; ++i) {
    const uint32_t v = lh[i * T + threadIdx.x];
    if (v) {
      atomicAdd(&dst[i * T + threadIdx.x], v);
      lh[i * T + threadIdx.x] = 0u;
    }
  }
  __syncthreads();
}

template <bool STATS, int GT, int T>
__global__ void __launch_bounds__(T)
k_small_step(SmallStep a) {
  constexpr int M = T == 1024 ? 2 : 4;
  constexpr int C = 8 * T, WAVES = T / 64, BPT = kHistBins / T;
  constexpr int POOL = C > kHistBins ? C : kHistBins;
  __shared__ __attribute__((aligned(16))) uint32_t pool[POOL];  // the block's histogram; at last its part of the update
  __shared__ uint16_t place[C];  // the chunk's kept elements, in order
  __shared__ SelState st;
  __shared__ uint32_t part[WAVES];
  __shared__ uint64_t wtot[WAVES];
  __shared__ double var_sh[STATS ? kMaxW : 1];
  __shared__ __attribute__((aligned(16))) uint32_t tail[128];
  __shared__ uint16_t owned[kSmallMaxChunks];
  __shared__ uint32_t few[kSmallFew];
  __shared__ int verdict;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t n = a.n;
  const int nchunks = a.nchunks, w_count = a.w_count, groups = a.groups, nunits = nchunks * groups, u0 = blockIdx.x;
  const SmallScratch& ss = a.ss;
  const bool known = a.leader >= 0;

  meet_start();
  // the first worker's loads are on their way while the chunk is taken
  v4f g8[2], r8[2];
  // the workers of a unit's group: a known leader alone in group 0 (as long as there are others), else shares of them all
  const int rest = w_count - 1;
  auto first_of = [&](int grp) __attribute__((always_inline)) {
    return known ? rest * (grp - 1) / (groups > 1 ? groups - 1 : 1) : w_count * grp / groups;
  };
  auto worker = [&](int i) __attribute__((always_inline)) { return known && i >= a.leader ? i + 1 : i; };
  auto fetch = [&](int w, int c) __attribute__((always_inline)) {
    small_fetch<GT>(a.g.p[w], a.res.p[w], n, (int64_t)c * C + 8 * tid, g8, r8);
  };
  auto fetch_first = [&](int unit) __attribute__((always_inline)) {
    const int grp = unit / nchunks;
    fetch(known && grp == 0 ? a.leader : worker(first_of(grp)), unit % nchunks);
  };
  fetch_first(u0);
  const uint32_t step = ss.ctr[kCtrStep];
  if (*a.err != 0u) return;  // (from before this launch, or set by a block of it that has given up: see meet_wait)
  const Meeting meet{ss.claim, ss.ctr + kCtrArrive + (step & 1u) * kCtrSet, step + 1u, nunits};
  if (tid == 0) {
    verdict = meet_take(meet, u0) ? 0 : -1;
    owned[0] = (uint16_t)u0;
  }
  for (int b = tid; b < kHistBins; b += T) pool[b] = 0u;
  if (tid < 128) tail[tid] = 0u;
  __syncthreads();
  // The step's number goes up once every block has read it: at once where every block took its own chunk, else when
  // as many blocks as chunks were taken on by others have come late, and this (the last to leave, then) is through.
  auto leave = [&](uint32_t helped) __attribute__((always_inline)) {
    if (tid != 0) return;
    bool last = true;
    if (helped != 0u) {
      const uint32_t late = __hip_atomic_fetch_add(&ss.ctr[kCtrLate], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      last = late == load_through(&ss.ctr[kCtrHelped]);
    }
    if (last) {
      store_through(&ss.ctr[kCtrStep], step + 1u);
      if (helped != 0u) {
        store_through(&ss.ctr[kCtrHelped], 0u);
        store_through(&ss.ctr[kCtrLate], 0u);
      }
    }
  };
  if (verdict < 0) return leave(1u);
  int n_owned = u0 < nchunks ? 1 : 0;  // chunks that this block takes to the outputs: of the first group

  uint32_t* const dig2 = ss.dig2 + (step & 1u) * kSmallReps * 128;

  uint32_t raw[8];  // the leader's elements of chunk `cur`
  int cur = -1;
  // acc = g + residual of worker w's chunk c, from what small_fetch has loaded; counts the top digits in `pool`
  auto sum_up = [&](int w, int c, const v4f (&ga)[2], const v4f (&ra)[2], VarAcc* va, bool count) __attribute__((always_inline)) {
    const int64_t j0 = (int64_t)c * C + 8 * tid;
    const bool full = j0 + 8 <= n;
    float* __restrict__ rp = a.res.p[w];
    v4f v[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      v[u].x = ga[u].x + ra[u].x;
      v[u].y = ga[u].y + ra[u].y;
      v[u].z = ga[u].z + ra[u].z;
      v[u].w = ga[u].w + ra[u].w;
    }
    if (full) {
      if (groups > 1) {  // (another block gathers from them)
#pragma unroll
        for (int u = 0; u < 4; ++u)
          store_through(reinterpret_cast<uint64_t*>(rp + j0) + u,
                        ((uint64_t)__float_as_uint(v[u >> 1][2 * (u & 1) + 1]) << 32) | __float_as_uint(v[u >> 1][2 * (u & 1)]));
      } else {
        store4<false>(rp + j0, v[0]);
        store4<false>(rp + j0 + 4, v[1]);
      }
      if (STATS) {
        va->seed4(a.raw_stats ? ga[0] : v[0]);
        va->add4(a.raw_stats ? ga[0] : v[0]);
        va->add4(a.raw_stats ? ga[1] : v[1]);
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if (j0 + e < n) {
          store_through(rp + j0 + e, v[e >> 2][e & 3]);
          if (STATS) {
            va->seed1(a.raw_stats ? ga[e >> 2][e & 3] : v[e >> 2][e & 3]);
            va->add1(a.raw_stats ? ga[e >> 2][e & 3] : v[e >> 2][e & 3]);
          }
        }
      }
    }
    if (count) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t bits = __float_as_uint(v[e >> 2][e & 3]);
        raw[e] = bits;
        if (full || j0 + e < n) atomicAdd(&pool[(bits & kKeyMask) >> 19], 1u);
      }
    }
  };
  // the first part of a chunk, its first worker's elements loaded already
  auto begin = [&](int unit) __attribute__((always_inline)) {
    const int c = unit % nchunks, grp = unit / nchunks;
    if (known && grp == 0) {
      sum_up(a.leader, c, g8, r8, nullptr, true);
      cur = c;
      small_flush<T>(pool, ss.hist + (size_t)(c % a.reps) * kHistBins);
    } else {
      const int end = first_of(grp + 1);
      for (int i = first_of(grp); i < end; ++i) {
        const int w = worker(i);
        const v4f ga[2] = {g8[0], g8[1]}, ra[2] = {r8[0], r8[1]};
        if (i + 1 < end) fetch(worker(i + 1), c);
        VarAcc va;
        sum_up(w, c, ga, ra, &va, !known);
        if (known) continue;
        if (STATS) block_moments<T, true>(va, a.partials, w, nchunks, c);
        small_flush<T>(pool, ss.hist + ((size_t)w * kSmallReps + (size_t)(c % a.reps)) * kHistBins);
      }
    }
    meet_arrive(meet, 0, unit);
  };
  // the sums of the workers other than a known leader, up to the upto-th of them
  int others = known && groups == 1 ? 0 : rest;
  auto more = [&](int upto) __attribute__((always_inline)) {
    while (others < upto) {
      const int m = upto - others < M ? upto - others : M;  // as many workers' loads in flight
      for (int i = 0; i < n_owned; ++i) {
        const int c = owned[i];
        const int64_t j0 = (int64_t)c * C + 8 * tid;
        v4f ga[M][2], ra[M][2];
#pragma unroll
        for (int q = 0; q < M; ++q) {
          if (q < m) {
            const int w = worker(others + q);
            small_fetch<GT>(a.g.p[w], a.res.p[w], n, j0, ga[q], ra[q]);
          }
        }
#pragma unroll
        for (int q = 0; q < M; ++q)
          if (q < m) sum_up(worker(others + q), c, ga[q], ra[q], nullptr, false);
      }
      others += m;
    }
  };

  begin(u0);
  if (n_owned == 0) return;
  more((rest + 2) / 3);
  for (int look = u0 + 1, looks = kHelpLooks; !meet_wait(meet, 0, nunits, looks, verdict); looks = 0) {
    const int c = meet_help(meet, look, &ss.ctr[kCtrHelped], verdict);
    if (c < 0) {  // all are taken, by blocks that run
      if (meet_wait(meet, 0, nunits, meet_limit(), verdict)) break;
      if (tid == 0) atomicOr(a.err, kErrWait);
      return;
    }
    look = c + 1;
    if (tid == 0 && c < nchunks) owned[n_owned] = (uint16_t)c;
    __syncthreads();
    fetch_first(c);
    begin(c);
    if (known && groups == 1) {  // (its share of what the other chunks have had of the other workers)
      for (int o = 0; o < others; ++o) {
        fetch(worker(o), c);
        sum_up(worker(o), c, g8, r8, nullptr, false);
      }
    }
    n_owned += c < nchunks ? 1 : 0;
  }

  // the leader
  int lead = a.leader;
  if (!known) {
    if (STATS) {
      for (int w = wave; w < w_count; w += WAVES) {
        const double v = wave_variance<true>(a.partials, w, nchunks);
        if (lane == 0) var_sh[w] = v;
      }
      __syncthreads();
      lead = 0;
      for (int w = 1; w < w_count; ++w)
        if (var_sh[w] > var_sh[lead]) lead = w;
      lead = __builtin_amdgcn_readfirstlane(lead);
    } else {
      lead = *a.leader_dev;
    }
  }
  const bool first = owned[0] == 0;  // chunk 0's block reports (or whoever took it, below)
  bool reports = first;
  for (int i = 1; i < n_owned; ++i) reports = reports || owned[i] == 0;
  if (reports) {
    if (STATS && !known && a.var_out && tid < w_count) a.var_out[tid] = var_sh[tid];
    if (tid == 0 && (known || STATS)) {
      *a.leader_dev = lead;
      if (a.leader_out) *a.leader_out = lead;
    }
    // the set of the next step (of the one before last: nobody is at it)
    uint32_t* const next = ss.ctr + kCtrArrive + ((step + 1u) & 1u) * kCtrSet;
    if (tid < 3 * kMeetWords) next[tid * kMeetLine] = 0u;
    for (int i = tid; i < kSmallReps * 128; i += T) ss.dig2[((step + 1u) & 1u) * kSmallReps * 128 + i] = 0u;
  }
  const float* lx = a.res.p[lead];

  // picks digit `digit` of the threshold from the counts in `pool`
  auto pick_here = [&](int digit) __attribute__((always_inline)) {
    __syncthreads();
    uint32_t h[BPT];
#pragma unroll
    for (int j = 0; j < BPT / 4; ++j) {
      uint4* const mine = reinterpret_cast<uint4*>(pool) + (BPT / 4) * tid + j;
      const uint4 q = *mine;
      h[4 * j + 0] = q.x;
      h[4 * j + 1] = q.y;
      h[4 * j + 2] = q.z;
      h[4 * j + 3] = q.w;
      *mine = make_uint4(0u, 0u, 0u, 0u);
    }
    block_pick_bins<T>(st, h, digit, part, a.err);
  };
  // the same from `reps` copies of its histogram
  auto pick = [&](const uint32_t* __restrict__ hist, auto digit_tag) __attribute__((always_inline)) {
    constexpr int digit = decltype(digit_tag)::value, pairs = (int)(digit_mask(digit) + 1u) / 2;
    // neighbouring lanes read neighbouring bins, all of a copy's loads together; `pool` hands them to the bins' owners
    constexpr int J = pairs > T ? pairs / T : 1;
    uint64_t sum[J];
#pragma unroll
    for (int j = 0; j < J; ++j) sum[j] = 0ull;
    for (int r = 0; r < a.reps; ++r) {
      const uint64_t* __restrict__ from = reinterpret_cast<const uint64_t*>(hist) + (size_t)r * pairs;
      uint64_t q[J];
#pragma unroll
      for (int j = 0; j < J; ++j) q[j] = pairs >= T || tid < pairs ? load_through(from + j * T + tid) : 0ull;
#pragma unroll
      for (int j = 0; j < J; ++j) sum[j] += q[j];
    }
#pragma unroll
    for (int j = 0; j < J; ++j)
      if (pairs >= T || tid < pairs) reinterpret_cast<uint64_t*>(pool)[j * T + tid] = sum[j];
    pick_here(digit);
  };
  // the leader's elements of chunk c in `raw`
  auto take = [&](int c) __attribute__((always_inline)) {
    if (c == cur) return;
    cur = c;
    const int64_t j0 = (int64_t)c * C + 8 * tid;
    if (groups > 1) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint64_t x = j0 + 2 * e + 2 <= n ? load_through(reinterpret_cast<const uint64_t*>(lx + j0) + e) : 0ull;
        raw[2 * e] = (uint32_t)x;
        raw[2 * e + 1] = (uint32_t)(x >> 32);
      }
      if (j0 < n && n - j0 < 8 && (n & 1)) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (j0 + e == n - 1) raw[e] = load_through(reinterpret_cast<const uint32_t*>(lx) + n - 1);
      }
    } else if (j0 + 8 <= n) {
      const uint4 x = reinterpret_cast<const uint4*>(lx + j0)[0], y = reinterpret_cast<const uint4*>(lx + j0)[1];
      raw[0] = x.x, raw[1] = x.y, raw[2] = x.z, raw[3] = x.w;
      raw[4] = y.x, raw[5] = y.y, raw[6] = y.z, raw[7] = y.w;
    } else if (j0 < n) {
#pragma unroll
      for (int e = 0; e < 8; ++e) raw[e] = __float_as_uint(lx[j0 + e < n ? j0 + e : n - 1]);
    }
  };
  if (!known) {
    cur = -1;
    take(owned[0]);
  }
  if (tid == 0) {
    st = SelState{};
    st.hi = kKeyMask;
    st.need = a.k;
  }
  pick(ss.hist + (known ? 0 : (size_t)lead * kSmallReps * kHistBins), std::integral_constant<int, 0>{});
  const uint32_t cand0 = st.cand, list0 = st.n_gt + st.cand;  // (reported)

  // every block has read the top digits' histograms; each clears its share
  auto clear_top = [&]() __attribute__((always_inline)) {
    uint4* __restrict__ z = reinterpret_cast<uint4*>(ss.hist);
    const int words4 = (known ? 1 : w_count) * kSmallReps * (kHistBins / 4);
    for (int i = 0; i < n_owned; ++i)
      for (int q = (int)owned[i] * T + tid; q < words4; q += nchunks * T) z[q] = make_uint4(0u, 0u, 0u, 0u);
  };
  uint32_t helped = 0u;  // (of the block that reports, thread 0; all chunks have been taken when it looks)
  auto last_wait = [&](int wait) __attribute__((always_inline)) {
    more(rest);
    if (reports && tid == 0) helped = load_through(&ss.ctr[kCtrHelped]);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (the block gathers from its workers' sums)
    const bool ok = meet_wait(meet, wait, nchunks, meet_limit(), verdict);
    if (!ok && tid == 0) atomicOr(a.err, kErrWait);
    return ok;
  };
  // Few candidates, all known when the top digits are: each chunk hands on its own instead of their digits' counts, and every
  // block picks both digits from them: one wait less, and no 16 KB to read (65537 x 2, one in a hundred, 570 candidates in
  // 17 chunks: 19.4 us with counts, 18.4 so with both digits counted on chip, 17.3 with the last from up to 64 keys in
  // registers and scans by lanes).  The line is where a chunk's share of `rows` takes all of them, whosever they are.
  const int row_words = kSmallRows / nchunks;
  const bool by_keys = nchunks <= kSmallFewChunks && cand0 < (uint32_t)row_words && cand0 <= (uint32_t)kSmallFew;
  uint32_t few_at = 0u, few_over = 0u;  // of chunk `lane`: its first candidate in `few`, and how many keys lie above them
  if (by_keys) {
    for (int i = 0; i < n_owned; ++i) {
      const int c = owned[i];
      take(c);
      const int64_t left = n - ((int64_t)c * C + 8 * tid);
      const uint32_t lo = st.lo, hi = st.hi;
      uint32_t is = 0u, up = 0u;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t kk = raw[e] & kKeyMask;
        up += e < left && kk > hi ? 1u : 0u;
        is |= e < left && kk >= lo && kk <= hi ? 1u << e : 0u;
      }
      const uint32_t cnt = (uint32_t)__popc(is);
      uint32_t at = 1u, tot = 0u;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const uint64_t pc = __ballot((cnt >> b) & 1u), pu = __ballot((up >> b) & 1u);
        at += popc_lt(pc) << b;
        tot += ((uint32_t)__popcll(pc) << b) + ((uint32_t)__popcll(pu) << (b + 16));
      }
      if (lane == 0) part[wave] = tot;
      __syncthreads();
      uint32_t sum = 0u;
#pragma unroll
      for (int v = 0; v < WAVES; ++v) {
        at += v < wave ? part[v] & 0xffffu : 0u;
        sum += part[v];
      }
      uint32_t* __restrict__ row = ss.rows + (size_t)c * row_words;
      if (tid == 0) store_through(row, sum);
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if ((is >> e) & 1u) store_through(row + at++, raw[e] & kKeyMask);
      meet_arrive(meet, 1, c);
    }
    if (!last_wait(1)) return;
    // (a row's first 64 candidates are on their way before it is known how many there are)
    constexpr int R = kSmallFewChunks / WAVES;
    const uint32_t head = lane < nchunks ? load_through(ss.rows + lane * row_words) : 0u;
    uint32_t q[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int c = wave + r * WAVES;
      q[r] = c < nchunks ? load_through(ss.rows + c * row_words + 1 + lane) : 0u;
    }
    const uint32_t have = (head & 0xffffu) < (uint32_t)row_words ? head & 0xffffu : 0u;
    few_over = head >> 16;
    few_at = wave_incl_scan(have) - have;
    auto put = [&](uint32_t at, uint32_t kk) __attribute__((always_inline)) {
      if (at < (uint32_t)kSmallFew) few[at] = kk;
      atomicAdd(&pool[(kk >> 7) & 0xfffu], 1u);
    };
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int c = wave + r * WAVES;
      if (c < nchunks) {
        const uint32_t cnt = (uint32_t)__builtin_amdgcn_readlane((int)have, c);
        const uint32_t at = (uint32_t)__builtin_amdgcn_readlane((int)few_at, c);
        if ((uint32_t)lane < cnt) put(at + lane, q[r]);
        for (uint32_t e = 64u + lane; e < cnt; e += 64u) put(at + e, load_through(ss.rows + c * row_words + 1 + e));
      }
    }
    pick_here(1);
    clear_top();
    const uint32_t lo = st.lo, hi = st.hi, left = st.cand, need = st.need;
    if (left <= 64u) {  // (nearly always: a lane takes one and counts those above and beside it)
      for (uint32_t e = (uint32_t)tid; e < cand0; e += T) {
        const uint32_t kk = few[e];
        if (kk >= lo && kk <= hi) {
          const uint32_t at = atomicAdd(&tail[64], 1u);
          if (at < 64u) tail[at] = kk;
        }
      }
      __syncthreads();
      if (wave == 0) {
        const bool real = (uint32_t)lane < left;
        const uint32_t mine = real ? tail[lane] : 0u;
        uint32_t over = 0u, same_key = 0u;
        for (int i = 0; i < (int)same(left); ++i) {
          const uint32_t x = (uint32_t)__builtin_amdgcn_readlane((int)mine, i);
          over += x > mine ? 1u : 0u;
          same_key += x == mine ? 1u : 0u;
        }
        const uint64_t hit = __ballot(real && over < need && need <= over + same_key);
        if (lane == 0 && hit == 0ull) atomicOr(a.err, kErrPick);
        if (hit != 0ull && lane == __builtin_ctzll(hit)) {
          st.lo = st.hi = mine;
          st.n_gt += over;
          st.need = need - over;
          st.cand = same_key;
          st.level = 3u;
        }
      }
      __syncthreads();
    } else {
      for (uint32_t e = (uint32_t)tid; e < cand0; e += T) {
        const uint32_t kk = few[e];
        if (kk >= lo && kk <= hi) atomicAdd(&pool[kk & 0x7fu], 1u);
      }
      pick_here(2);
    }
  } else {
    for (int i = 0; i < n_owned; ++i) {
      const int c = owned[i];
      take(c);
      const int64_t left = n - ((int64_t)c * C + 8 * tid);
      const uint32_t lo = st.lo, hi = st.hi;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t kk = raw[e] & kKeyMask;
        if (e < left && kk >= lo && kk <= hi) atomicAdd(&pool[(kk >> 7) & 0xfffu], 1u);
      }
      small_flush<T>(pool, ss.dig1 + (size_t)(c % a.reps) * kHistBins);
      meet_arrive(meet, 1, c);
    }
    more((2 * rest + 2) / 3);
    if (!meet_wait(meet, 1, nchunks, meet_limit(), verdict)) {
      if (tid == 0) atomicOr(a.err, kErrWait);
      return;
    }
    pick(ss.dig1, std::integral_constant<int, 1>{});

    for (int i = 0; i < n_owned; ++i) {
      const int c = owned[i];
      take(c);
      const int64_t left = n - ((int64_t)c * C + 8 * tid);
      const uint32_t lo = st.lo, hi = st.hi;
      uint32_t up = 0u;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t kk = raw[e] & kKeyMask;
        up += e < left && kk > hi ? 1u : 0u;
        if (e < left && kk >= lo && kk <= hi) atomicAdd(&tail[kk & 0x7fu], 1u);
      }
      uint32_t all = 0u;
#pragma unroll
      for (int b = 0; b < 4; ++b) all += (uint32_t)__popcll(__ballot((up >> b) & 1u)) << b;
      if (lane == 0) part[wave] = all;
      __syncthreads();
      if (wave == 0) {  // lane's digits 2 lane and 2 lane + 1
        const uint32_t t0 = tail[2 * lane], t1 = tail[2 * lane + 1];
        uint32_t* __restrict__ d2 = dig2 + (size_t)(c % a.reps) * 128;
        if (t0) atomicAdd(&d2[2 * lane], t0);
        if (t1) atomicAdd(&d2[2 * lane + 1], t1);
        const uint32_t incl = wave_incl_scan(t0 + t1);
        const uint32_t s = wave_last(incl) - incl + t0 + t1;
        store_through(reinterpret_cast<uint64_t*>(ss.rows + (size_t)c * 128) + lane, ((uint64_t)(s - t0) << 32) | s);
        tail[2 * lane] = tail[2 * lane + 1] = 0u;
        if (lane == 0) {
          uint32_t sum = 0u;
#pragma unroll
          for (int v = 0; v < WAVES; ++v) sum += part[v];
          store_through(&ss.above[c], sum);
        }
      }
      meet_arrive(meet, 2, c);
    }
    clear_top();
    if (!last_wait(2)) return;
    pick(dig2, std::integral_constant<int, 2>{});
  }
  if (reports && tid == 0) {
    SelState out = st;
    out.many = cand0 > small_few(n) ? 1u : 0u;
    out.compact_level = list0 <= a.list_cap ? 1u : 0u;
    out.list_count = out.compact_level ? list0 : 0u;
    *a.st = out;
    if (st.level != 3u) atomicOr(a.err, kErrSequence);
  }
  if (!by_keys) {
    uint4* __restrict__ z = reinterpret_cast<uint4*>(ss.dig1);
    for (int i = 0; i < n_owned; ++i)
      for (int q = (int)owned[i] * T + tid; q < kSmallReps * (kHistBins / 4); q += nchunks * T)
        z[q] = make_uint4(0u, 0u, 0u, 0u);
  }
  if (reports) leave(helped);
  if (st.level != 3u) return;

  const uint32_t klo = st.lo, khi = st.hi, quota = st.need, digit = klo & 0x7fu;
  float* const buf = reinterpret_cast<float*>(pool);
  for (int i = 0; i < n_owned; ++i) {
    const int c = owned[i];
    // kept in front of the chunk: keys above the threshold, and at it
    uint64_t before = 0ull;
    if (by_keys) {
      if (tid < c) before = (uint64_t)few_over << 32;  // (fewer chunks than a wave has lanes)
      const uint32_t upto = (uint32_t)__builtin_amdgcn_readlane((int)few_at, same(c));
      for (uint32_t e = (uint32_t)tid; e < upto && e < (uint32_t)kSmallFew; e += T)
        before += few[e] > khi ? 1ull << 32 : few[e] >= klo ? 1ull : 0ull;
    } else if (tid < c) {
      const uint32_t* __restrict__ row = ss.rows + (size_t)tid * 128 + digit;
      const uint32_t at = load_through(row), over = digit < 127u ? load_through(row + 1) : 0u;
      before = ((uint64_t)(load_through(&ss.above[tid]) + over) << 32) | (at - over);
    }
    take(c);
    const int64_t left = n - ((int64_t)c * C + 8 * tid);
    uint32_t isA = 0u, isB = 0u;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint32_t kk = raw[e] & kKeyMask;
      isA |= e < left && kk > khi ? 1u << e : 0u;
      isB |= e < left && kk >= klo && kk <= khi ? 1u << e : 0u;
    }
    const uint32_t cA = (uint32_t)__popc(isA), cB = (uint32_t)__popc(isB);
    uint32_t bA = 0u, bB = 0u, totA = 0u, totB = 0u;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const uint64_t pa = __ballot((cA >> b) & 1u), pb = __ballot((cB >> b) & 1u);
      bA += popc_lt(pa) << b;
      bB += popc_lt(pb) << b;
      totA += (uint32_t)__popcll(pa) << b;
      totB += (uint32_t)__popcll(pb) << b;
    }
    before = wave_allsum_u64(before);
    __syncthreads();  // (wtot, var_sh's and the last chunk's uses of `pool` are over)
    if (lane == 0) {
      wtot[wave] = ((uint64_t)totA << 32) | totB;
      reinterpret_cast<uint64_t*>(tail)[wave] = before;
    }
    for (int b = tid; b < C / 4; b += T) reinterpret_cast<uint4*>(pool)[b] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    uint64_t front = 0ull, mine = 0ull, chunk = 0ull;
#pragma unroll
    for (int v = 0; v < WAVES; ++v) {
      front += reinterpret_cast<const uint64_t*>(tail)[v];
      mine += v < wave ? wtot[v] : 0ull;
      chunk += wtot[v];
    }
    auto kept = [&](uint64_t ab) __attribute__((always_inline)) {
      const uint32_t b = (uint32_t)ab;
      return (uint32_t)(ab >> 32) + (b < quota ? b : quota);
    };
    const uint32_t m0 = kept(front), m1 = kept(front + chunk);
    bA += (uint32_t)((front + mine) >> 32);
    bB += (uint32_t)(front + mine);
    if ((isA | isB) != 0u) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const bool is_a = (isA >> e) & 1u, is_b = (isB >> e) & 1u;
        if (is_a || (is_b && bB < quota)) place[bA + (bB < quota ? bB : quota) - m0] = (uint16_t)(8 * tid + e);
        bA += is_a ? 1u : 0u;
        bB += is_b ? 1u : 0u;
      }
    }
    __syncthreads();
    for (uint32_t q = (uint32_t)tid; q < m1 - m0; q += T) {
      const uint32_t at = place[q], m = m0 + q;
      const int64_t j = (int64_t)c * C + at;
      if (m >= a.k) break;
      float s = 0.0f;
      for (int w0 = 0; w0 < w_count; w0 += 8) {  // eight independent loads in flight, then the ordered adds
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (w0 + u < w_count) v[u] = groups > 1 ? load_through(a.res.p[w0 + u] + j) : a.res.p[w0 + u][j];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          if (w0 + u < w_count) {
            if (a.vals) a.vals[(size_t)(w0 + u) * (size_t)a.k + (size_t)m] = v[u];
            s = w0 + u == 0 ? v[u] : s + v[u];
            a.res.p[w0 + u][j] = 0.0f;
          }
        }
      }
      a.idx_out[m] = (int32_t)j;
      a.sum_out[m] = s;
      buf[at] = s;
    }
    if (a.update == nullptr) continue;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int at = 4 * (u * T + tid);
      const int64_t j = (int64_t)c * C + at;
      if (j + 4 <= n) {
        store4<false>(a.update + j, reinterpret_cast<const v4f*>(pool)[u * T + tid]);
      } else {
        for (int e = 0; j + e < n; ++e) a.update[j + e] = buf[at + e];
      }
    }
  }
}

}  // namespace artopk
