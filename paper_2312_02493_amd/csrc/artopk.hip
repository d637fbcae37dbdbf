// Host side of the AR-Topk compressor library: argument checks, scratch
// management and kernel sequencing behind the C ABI declared in artopk.h.
// No call synchronises the stream except artopk_status / artopk_get_profile /
// artopk_destroy; all decisions that depend on the data (leader, thresholds,
// tie quotas, list sizes) stay in device memory.

#include "artopk.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "artopk_kernels.h"

using namespace artopk;

// Fixed scratch of artopk_variance_static (the entry point that allocates nothing): the per-block
// moments of up to kMaxW workers x kMaxChunks blocks, then kMaxW variances, then the argmax word.
// Every GPU the library runs on holds its own copy until the process ends.  In host code this name
// is only a handle for hipGetSymbolAddress; the kernels get the address that call returns.
constexpr size_t kStaticPartials = (size_t)kMaxW * kMaxChunks * 3;
constexpr size_t kStaticDoubles = kStaticPartials + kMaxW + 1;
static __device__ __align__(256) double scratch[kStaticDoubles];

namespace {

constexpr int kPassAThreads = 1024, kPassAU = 8;        // 128 KiB of each array per block iteration
constexpr int kPassRestThreads = 1024, kPassRestU = 8;

constexpr int32_t kMaxBatch = 16;  // vectors selected on in one launch set
// Default of ARTOPK_OPT_GUESS_MIN_N, and what stands in its place for vectors that are only read: elements of
// the vectors selected on together.  Measured (us, histogram route / read-only marking, one in a thousand, a hundred
// and 33 kept, heavy tails): 1 x 12 M 60/60 61/64 64/70, 16.8 M 67/63 70/67 71/75, 20 M 79/68 82/70 85/82, 23 M 81/68
// 86/73 88/84, 25.6 M 90/71 92/77 99/90; 2 x 10 M 86/77 88/81 93/92; 4 x 5 M 82/80 85/86; 8 x 2.5 M 86/84 90/89, 4 M
// 116/97 119/102; 16 x 1.5 M 98/108.  The line lies where all of them gain.  (One in ten kept: 25.6 M 116 against 137,
// 138 M 390 against 389, so denser than one in 32 never.)
constexpr int64_t kGuessMinN = (int64_t)1 << 25, kReadGuessMinN = (int64_t)3 << 23;
constexpr int64_t kTwiceMaxN = (int64_t)5 << 23;  // (see plan_guess_read)

// Flat steps on short vectors run in one launch (small_step) up to ARTOPK_OPT_SHORT_MAX_N elements, or three quarters
// of that where the leader is found on the device and fewer than eight workers share the cost of that.  Measured, us, ten
// or eight launches / one, one in a hundred kept, 786427, 1 M, 1.3 M and 1.8 M elements: leader known, 2 workers 59/25
// 59/28 60/28 63/31, 4 workers 61/24 62/26 65/29 69/33, 8 workers 64/29 67/33 76/40 84/47, 16 workers 80/43 87/49 98/60
// 117/72; variance rule, 2 workers 52/32 53/36 60/39 -, 4 workers 62/38 65/41 73/48 -, 8 workers 77/50 87/53 97/68
// 117/75, 16 workers 114/77 133/79 152/105 189/113.  So both lines lie below the crossing, which is beyond 1.8 M for all of
// these: they are those of the option's documented default, where the short vectors' launches used to cross, and a caller
// who sets the option has the launch up to 2^21.  Any number kept: a tenth, a third and all of 65537 x 2 63/21 71/21 90/23, of 1 M x 8 75/38
// 90/39 118/40; variance rule, 65537 x 8 53/39 57/41 67/44, 1 M x 8 94/59 103/62 117/59.
constexpr int64_t kSmallMaxN = (int64_t)1 << 20, kSmallMaxNLimit = (int64_t)kSmallMaxChunks * kTile;
// Where the leader comes from statistics, a block takes its chunk of one worker after the other, and beyond this many values
// of more than 24 workers the general launches are ahead on vectors whose chunks do not fill the chip, unless the option
// was set.  One launch / eight, us, one in a hundred and in ten kept: 524288 x 48 144/148 167/145, x 64 185/182 215/180,
// 700001 x 32 134/127 170/147, x 48 190/170 244/196, 786427 x 32 137/126 176/145, x 64 255/215 332/252; outside 700001 x 24
// 107/108 133/128, 400009 x 64 159/175 190/168, and with all the chip 1 M x 32 128/142 182/168.
constexpr int64_t kSmallMaxValues = 22000000, kSmallManyMinN = (int64_t)1 << 19, kSmallManyMaxN = (int64_t)3 << 18;

// Selections by tiles from this many elements on: flat ones of a leader known up front.  Launches of the histogram route /
// tiles, us, one in a hundred and in ten kept, 3 M x 2 73/81 86/94, 6 M x 2 93/93 118/110, x 8
// 171/172 198/193, 12 M x 2 125/120 153/144, x 8 273/268 312/294, 25.6 M x 2 218/193 291/227, bfloat16 gradients 12 M x 8
// 236/237 280/268, 25.6 M x 8 449/427 550/478.
constexpr int64_t kTilesMinN = (int64_t)3 << 22;

// Segmented selections by tiles (segments_by_tiles).  List kernels / tiles, us, a selection, one in a hundred kept; s: in as
// many equal segments, u: of sizes spread over a factor of 40,000.
//   Every segment costs a sample, a pick and tiles that are not whole, the list kernels more the longer the longest one is:
// 8.4 M u2 69/61, u8 69/60, s3 59/65, u20 63/64, u54 64/76, u250 76/96; 10 M s3 69/63, u20 64/65, u54 67/69; 12.6 M s3 71/64,
// u20 70/67, u54 68/82, u250 90/100; 16 M u54 81/72, u100 85/90, u160 108/95, u250 95/105; 20 M u54 90/89, u250 101/106; 25.6 M
// u54 110/80, u700 154/147.
//   A segment without pieces is read by each of the kernels behind the marking, the parts of a block's four tiles one after
// the other, and then the more the longer it is.  One such segment among four, of 512 / 2048 / 16384 / 32768 elements, 16 M
// 72/74 72/82 72/88 73/108, 25.6 M 105/84 106/92 106/97 107/118; one in five kept of an eighth / a quarter / all of the
// elements, else one in a hundred, 25.6 M s8 111/171 117/178 143/202, 138 M 364/336 376/382 507/755; three in ten / four in
// ten kept, 25.6 M s8 174/210 200/202, 60 M s8 327/343 379/329, 138 M 704/783 826/773.  But the list kernels are slow where
// one segment is much longer than the others, or there are very many: three in ten, 25.6 M u54 276/203, s770 221/204, 138 M
// u54 1260/787, u1000 1173/760, s4000 1129/903.
constexpr int64_t kSegTilesMinN = (int64_t)1 << 23, kSegTilesSomeN = (int64_t)10 << 20, kSegTilesAllN = (int64_t)14 << 20;
constexpr int64_t kSegTilesBareN = (int64_t)3 << 23, kSegTilesFewBareN = (int64_t)3 << 25, kShortBare = 1024;
constexpr int32_t kSegTilesEach = 24, kSegTilesFew = 6, kSegTilesMany = 512;

struct Scratch {
  // zeroed before every select: one kSegWords block per segment, then the look-back flags
  uint32_t* h_all = nullptr;      // [max_w][kSlotWords] whole-vector histograms of the fused pass, guess sample
  uint64_t* mask = nullptr;       // [max_w][mask_stride] survivor bit masks of the fused pass
  int64_t mask_stride = 0;        // 64-bit words per worker
  uint32_t* zero_base = nullptr;  // [max_seg][kSegWords]
  uint64_t* flags = nullptr;      // [max_tiles][kNumLookback], directly behind the blocks
  int64_t max_tiles = 0;
  // not zeroed
  uint32_t* S = nullptr;          // [max_w * kMaxChunks + max_seg][4096] per-chunk suffix histograms
  uint32_t* chunk_off = nullptr;  // [16 kMaxChunks + max_seg]
  double* partials = nullptr;     // [max_w][kMaxPassBlocks][3] per-block moments (or [2] sums)
  double* var_scratch = nullptr;  // [max_w]
  int32_t* leader_dev = nullptr;
  uint64_t* counter_dev = nullptr;  // iteration counter of ARTOPK_STAR_COUNTER steps
  uint32_t* err_dev = nullptr;
  uint2* list = nullptr;          // survivor lists: (index, raw float bits)
  int64_t list_entries = 0;       // allocated entries
  float* vals = nullptr;          // [max_w][max_k] gathered rows when the caller passes no vals_out
  int32_t* idx_rows = nullptr;    // [max_w][max_k] every worker's own Top-k (literal Alg. 1 leader rule)
  int32_t* tile_start = nullptr;  // [max_n / kPassTile + 2] kept indices below every tile of the streaming pass
  uint2* tilebuf = nullptr;       // pieces of marked elements, of tiles or of the spans of vectors that are only read
  int64_t tilebuf_entries = 0;
  SmallScratch small{};           // short vectors' steps
  size_t small_words = 0;         // of it, zero whenever no step is running
  SegDesc* table_dev = nullptr;   // [max_seg] segment descriptors
  uint32_t* chunk_map = nullptr;  // [kMaxChunks + max_seg] (segment << 16) | chunk, one entry per chunk of the layout
  uint4* tile_map = nullptr;      // [map_tiles] tiles of a segmented layout, then their groups (TileArgs::map, groups)
  int64_t map_tiles = 0;
  uint32_t cap = 0;               // list capacity of a flat (one-segment) select
};

// A selection problem laid out for the kernels: one descriptor per segment and
// the launch bounds derived from them.
struct Plan {
  int32_t nseg = 1;
  std::vector<SegDesc> desc;
  bool use_table = false;   // descriptors live in the device table (nseg > 1)
  int32_t max_chunks = 1;   // largest chunk count of a segment
  int64_t max_tiles = 1;    // largest look-back tile count of a segment
  int64_t total_tiles = 1;
  int64_t max_cap = 1;      // largest list capacity of a segment
  int64_t k_all = 0;        // entries kept of all segments together
  size_t hist_words = 0;    // words of h_all's memory used for copies of histograms
  bool batch = false;       // nseg whole vectors with one descriptor (SelParams::batch)
  bool lists = false;       // select with the list kernels
  int64_t list_stride = 0;  // list entries per vector of a batch
  int32_t total_chunks = 0; // chunks of all segments together (entries of the device chunk map), 0: no map
  int32_t tiles = 0, tile_groups = 0;  // tiles of all segments together, 0: not selected on by tiles
  int32_t more_bins = 0;               // further copies of segments' bins
  bool tiles_aligned = true;           // they are the streaming passes' tiles
  int64_t longest = 0;   // elements of the longest segment,
  int64_t bare = 0;      // of those of more than a tile whose tiles will have no pieces,
  bool some_bare = false;  // and whether there are such of more than kShortBare
};

}  // namespace

struct artopk_ctx {
  int device = 0;
  int num_cu = 256;
  hipStream_t stream = nullptr;
  int32_t max_w = 0;
  int64_t max_n = 0, max_k = 0;
  int32_t max_seg = 0;
  bool pass_a_nt = true;   // non-temporal g loads / acc stores in pass A
  bool leader_first = true;  // STAR / FIXED: leader pass + select first, then one fused pass over the rest
  // vectors of at least this many elements get a sampled threshold guess before the fused pass, which
  // then counts and marks only the keys that reach it (the selection no longer re-reads the vector)
  int64_t guess_min_n = kGuessMinN;
  bool guess_min_n_set = false;  // by artopk_set_option: then it holds for vectors that are only read, too
  // vectors of at least this many elements get their dense update from k_update_tiles
  int64_t update_tiles_min_n = (int64_t)1 << 22;
  int stage_tiles = 1;  // marked elements are handed on by tiles: 0 never, 1 where that is the better way, 2 (flat vectors)
                        // whenever a piece can hold a tile's share
  int64_t small_max_n = kSmallMaxN;  // flat steps of up to about this many elements run in one launch
  bool small_max_n_set = false;      // by artopk_set_option: then however many workers there are
  void* slab = nullptr;
  Scratch s;
  // how the last step or selection ran (artopk_select_info)
  int32_t last_guessed = 0, last_dom_workers = 0, last_short = 0, last_one_launch = 0;
  int32_t last_tiles = 0;  // segments selected on by tiles (1: a flat vector), or 0
  int g_type = ARTOPK_G_F32;  // element type of the gradients of the step being enqueued
  // descriptors of the last segmented layout uploaded to table_dev
  std::vector<int64_t> cached_off, cached_k;
  int64_t cached_n = -1;
  Plan cached_plan;
  bool cached_map = false;  // the map of its tiles is made
  // stage events: a ring of the most recent calls, 5 marks per call
  // (0 start, 1 after pass A, 2 after select, 3 after gather, 4 after update)
  bool profile = false;
  int profile_level = 0;
  int lvl1_a = 0, lvl1_b = 1;  // the two marks level 1 records (they bracket the dominant kernel)
  static constexpr int kRing = 64;
  static constexpr int kMarks = 5;
  hipEvent_t ev[kRing][kMarks] = {};
  bool ev_valid[kRing][kMarks] = {};
  bool ev_created = false;
  long prof_calls = 0;  // calls recorded since profiling was switched on
  int cur = 0;          // ring slot of the call being recorded
  char err[512] = {0};
};
static_assert(sizeof(artopk_ctx::err) == 512, "fail() writes up to 512 bytes");

namespace {

// error text of calls that have no context (artopk_last_error(NULL) returns it)
thread_local char g_noctx_err[512] = {0};

int fail(artopk_ctx* c, int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(c ? c->err : g_noctx_err, sizeof(g_noctx_err), fmt, ap);
  va_end(ap);
  return code;
}

#define HIP_TRY(ctx, expr)                                                                   \
  do {                                                                                       \
    hipError_t e_ = (expr);                                                                  \
    if (e_ != hipSuccess)                                                                    \
      return fail((ctx), ARTOPK_EHIP, "%s failed: %s (%s:%d)", #expr, hipGetErrorString(e_), \
                  __FILE__, __LINE__);                                                       \
  } while (0)

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int check_ptr_table(artopk_ctx* c, const float* const* tab, int32_t w, const char* name, int align = 16) {
  if (!tab) return fail(c, ARTOPK_EINVAL, "%s is NULL", name);
  for (int i = 0; i < w; ++i) {
    if (!tab[i]) return fail(c, ARTOPK_EINVAL, "%s[%d] is NULL", name, i);
    if (reinterpret_cast<uintptr_t>(tab[i]) % (uintptr_t)align)
      return fail(c, ARTOPK_EINVAL, "%s[%d] is not %d-byte aligned", name, i, align);
  }
  return ARTOPK_OK;
}

int check_common(artopk_ctx* c, int32_t w, int64_t n, int64_t k) {
  if (!c) return ARTOPK_EINVAL;
  if (w < 1 || w > c->max_w) return fail(c, ARTOPK_EINVAL, "W=%d outside [1, %d]", w, c->max_w);
  if (n < 1 || n > c->max_n) return fail(c, ARTOPK_EINVAL, "N=%lld outside [1, %lld]", (long long)n, (long long)c->max_n);
  if (n >= (1ll << 31)) return fail(c, ARTOPK_EINVAL, "N must be below 2^31");
  if (k < 1 || k > n) return fail(c, ARTOPK_EINVAL, "k=%lld outside [1, N]", (long long)k);
  if (k > c->max_k) return fail(c, ARTOPK_EINVAL, "k=%lld above max_k=%lld", (long long)k, (long long)c->max_k);
  return ARTOPK_OK;
}

int check_segments(artopk_ctx* c, int64_t n, int32_t nseg, const int64_t* seg_off, const int64_t* seg_k,
                   int64_t k) {
  if (nseg < 1) return fail(c, ARTOPK_EINVAL, "nseg must be >= 1");
  if (nseg > c->max_seg) return fail(c, ARTOPK_EINVAL, "nseg=%d above max_segments=%d", nseg, c->max_seg);
  if ((seg_off == nullptr) != (seg_k == nullptr))
    return fail(c, ARTOPK_EINVAL, "seg_off and seg_k must both be given or both be NULL");
  if (!seg_off) {
    if (nseg != 1) return fail(c, ARTOPK_EINVAL, "nseg > 1 needs seg_off and seg_k");
    return ARTOPK_OK;
  }
  if (seg_off[0] != 0 || seg_off[nseg] != n) return fail(c, ARTOPK_EINVAL, "segments must cover [0, N)");
  int64_t ksum = 0;
  for (int s = 0; s < nseg; ++s) {
    const int64_t sz = seg_off[s + 1] - seg_off[s];
    if (sz < 1) return fail(c, ARTOPK_EINVAL, "segment %d is empty or descending", s);
    if (seg_k[s] < 1 || seg_k[s] > sz) return fail(c, ARTOPK_EINVAL, "seg_k[%d] outside [1, size]", s);
    ksum += seg_k[s];
  }
  if (ksum != k) return fail(c, ARTOPK_EINVAL, "sum of seg_k (%lld) differs from k (%lld)", (long long)ksum, (long long)k);
  return ARTOPK_OK;
}

// The buffers of one call as byte ranges.  Ranges that are only read may overlap each other
// (two workers may share a gradient buffer); a range that is written must not overlap any other.
class RangeSet {
 public:
  void add(const void* p, size_t bytes, bool written, const char* name, int index = -1) {
    if (!p || bytes == 0 || n_ >= kCap) return;
    const uintptr_t lo = reinterpret_cast<uintptr_t>(p);
    r_[n_++] = Range{lo, lo + bytes, written, name, index};
  }
  void add_table(const void* const* tab, int32_t w, size_t bytes, bool written, const char* name) {
    for (int i = 0; i < w; ++i) add(tab[i], bytes, written, name, i);
  }
  // ARTOPK_OK, or ARTOPK_EINVAL with the first offending pair in the context's error text
  int check(artopk_ctx* c) {
    std::sort(r_, r_ + n_, [](const Range& a, const Range& b) { return a.lo < b.lo; });
    int far_any = -1, far_written = -1;  // ranges seen so far that reach furthest: any, written ones
    for (int i = 0; i < n_; ++i) {
      const int other = r_[i].written ? far_any : far_written;
      if (other >= 0 && r_[i].lo < r_[other].hi) {
        char a[48], b[48];
        label(r_[other], a, sizeof(a));
        label(r_[i], b, sizeof(b));
        return fail(c, ARTOPK_EINVAL, "buffers %s and %s overlap", a, b);
      }
      if (far_any < 0 || r_[i].hi > r_[far_any].hi) far_any = i;
      if (r_[i].written && (far_written < 0 || r_[i].hi > r_[far_written].hi)) far_written = i;
    }
    return ARTOPK_OK;
  }

 private:
  struct Range {
    uintptr_t lo, hi;
    bool written;
    const char* name;
    int index;
  };
  static void label(const Range& r, char* out, size_t cap) {
    if (r.index >= 0)
      snprintf(out, cap, "%s[%d]", r.name, r.index);
    else
      snprintf(out, cap, "%s", r.name);
  }
  static constexpr int kCap = 2 * kMaxW + 8;
  Range r_[kCap];
  int n_ = 0;
};

PtrTable make_table(const float* const* tab, int32_t w) {
  PtrTable t;
  for (int i = 0; i < kMaxW; ++i) t.p[i] = (i < w) ? const_cast<float*>(tab[i]) : nullptr;
  return t;
}

// Chunk layout of the element range [e_lo, e_hi): at most max_chunks chunks of
// whole tiles, chunk 0 starting at the tile boundary at or below e_lo.
ChunkGeom make_geom(int64_t e_lo, int64_t e_hi, int64_t max_chunks = kMaxChunks, bool whole_pass_tiles = false) {
  ChunkGeom g;
  g.chunk0 = e_lo / kTile * kTile;
  const int64_t span = e_hi - g.chunk0;
  int64_t ce = (span + max_chunks - 1) / max_chunks;
  ce = (ce + kTile - 1) / kTile * kTile;
  if (ce < kTile) ce = kTile;
  // chunks longer than one tile of the fused pass are whole tiles of it, so that only the last
  // chunk of a vector has a ragged tile
  // (and always, if the pass strides over its tiles and counts per chunk)
  constexpr int64_t pass_tile = (int64_t)kPassAThreads * kPassAU * 4;
  static_assert(pass_tile == kPassTile, "the kernels' tile");
  if (ce > kTile || whole_pass_tiles) ce = (ce + pass_tile - 1) / pass_tile * pass_tile;
  g.chunk_elems = ce;
  g.nchunks = (int32_t)((span + ce - 1) / ce);
  if (g.nchunks < 1) g.nchunks = 1;
  return g;
}

// Blocks per worker of the stand-alone variance kernel.
int stats_blocks(int num_cu, int32_t w, int64_t n) {
  const int64_t n4 = n >> 2;
  const int64_t tile = 256 * kPassAUnroll;
  int64_t ntile = (n4 + tile - 1) / tile;
  if (ntile < 1) ntile = 1;
  int64_t want = ((int64_t)num_cu * 8 + w - 1) / w;
  if (want < 1) want = 1;
  int64_t nblk = ntile < want ? ntile : want;
  if (nblk > kMaxChunks) nblk = kMaxChunks;
  return (int)nblk;
}

// Beyond twice the last-level cache (256 MiB) reads of w vectors of n elements are non-temporal (see k_stats).
bool beyond_cache(int32_t w, int64_t n) { return (int64_t)w * n * 4 > ((int64_t)1 << 29); }

// Launches the statistics of w vectors of n elements (k_stats; rows 16-byte aligned).
void launch_stats(hipStream_t st, const PtrTable& x, int nblk, int32_t w, int64_t n, double* partials) {
  if (beyond_cache(w, n))
    hipLaunchKernelGGL(k_stats<true>, dim3(nblk, w), dim3(256), 0, st, x, n, partials);
  else
    hipLaunchKernelGGL(k_stats<false>, dim3(nblk, w), dim3(256), 0, st, x, n, partials);
}

// A stage boundary (level 2 only).
void prof_mark(artopk_ctx* c, int mark) {
  if (!c->profile || c->profile_level < 2) return;
  if (hipEventRecord(c->ev[c->cur][mark], c->stream) == hipSuccess) c->ev_valid[c->cur][mark] = true;
}

// Level 1: the two events directly around the launch of the step's dominant kernel, stored as the
// marks lvl1_a / lvl1_b so that they read as that kernel's stage.
void prof_dom(artopk_ctx* c, bool end) {
  if (!c->profile || c->profile_level != 1) return;
  const int mark = end ? c->lvl1_b : c->lvl1_a;
  if (hipEventRecord(c->ev[c->cur][mark], c->stream) == hipSuccess) c->ev_valid[c->cur][mark] = true;
}

// Starts the record of a new call in the next ring slot.
void prof_begin(artopk_ctx* c) {
  if (!c->profile) return;
  c->cur = (int)(c->prof_calls % artopk_ctx::kRing);
  c->prof_calls++;
  for (int i = 0; i < artopk_ctx::kMarks; ++i) c->ev_valid[c->cur][i] = false;
}

int64_t tiles_of_range(int64_t e_lo, int64_t e_hi) {
  return (e_hi + kCompactTile - 1) / kCompactTile - e_lo / kCompactTile;
}

int64_t seg_list_cap(int64_t n_s, int64_t k_s) {
  int64_t share = n_s / 8;
  if (share < 4096) share = 4096;
  int64_t cap = k_s + share;
  return cap < n_s ? cap : n_s;
}

// k_hist0's blocks add their occupied bins to a histogram of the range at about 0.1 us for each
// same-address atomic: a range of many chunks spreads them over kHistReps copies, which cost the pick
// about 4 us more to add up (eight selections on 25.6 M elements, 780 chunks: 0.88 ms with copies, 1.14
// without; one on 138 M, 845 chunks: no difference.  Segments of up to 128 chunks: 5 us slower with them).
constexpr int32_t kManyChunks = 128;

// List capacity of a flat selection whose list has `room` entries of memory.
int64_t vec_cap(const artopk_ctx* c, int64_t room) { return room < (int64_t)c->s.cap ? room : (int64_t)c->s.cap; }

// One segment covering the whole vector.  own_hist: no fused pass has built its histograms.
Plan flat_plan(const artopk_ctx* c, int64_t n, int64_t k, int32_t vec = -1, bool whole_pass_tiles = false,
               bool own_hist = false, int64_t max_chunks = kMaxChunks) {
  Plan pl;
  pl.nseg = 1;
  SegDesc d{};
  d.e_lo = 0;
  d.e_hi = n;
  d.geom = make_geom(0, n, max_chunks, whole_pass_tiles);
  d.koff = 0;
  d.list_base = 0;
  d.flag_base = 0;
  d.chunk_begin = 0;
  d.k = (uint32_t)k;
  d.cap = c->s.cap < (uint64_t)n ? c->s.cap : (uint32_t)n;
  d.vec = vec;
  d.hreps = own_hist && d.geom.nchunks > kManyChunks ? kHistReps : 1;
  d.tile_begin = 0;
  d.ntiles = (int32_t)((n + kMarkTile - 1) / kMarkTile);
  d.group_begin = d.bins_begin = 0;
  d.bins_more = 7;
  pl.k_all = k;
  pl.hist_words = d.hreps > 1 ? (size_t)d.hreps * kHistBins : 0;
  pl.desc.push_back(d);
  pl.max_chunks = d.geom.nchunks;
  pl.max_tiles = pl.total_tiles = tiles_of_range(0, n);
  pl.max_cap = d.cap;
  return pl;
}

// TileArgs' tables, one behind the other: where each begins, in words for every tile (kept has two of 64 bits: a tile's, and
// there are no more blocks than tiles), and where the further copies of segments' bins lie behind them all.
constexpr int kTileHeldAt = 4, kTileMarkedAt = kTileHeldAt + 1, kTileAboveAt = kTileMarkedAt + 1;
constexpr int kTileAmongAt = kTileAboveAt + kTileWaves, kTileSlotsAt = kTileAmongAt + kTileWaves;
constexpr int kTileWords = kTileSlotsAt + kTileSlots * kTileWaves;
static_assert((((int64_t)1 << 31) / kMarkTile + 2) * kTileWords < (int64_t)kMaxChunks * kHistBins,
              "one worker's S has room for them (that of each segment takes its two tiles more)");
static_assert(2 * kTileWords < kHistBins, "see there");
uint32_t* tile_more_bins(const artopk_ctx* c, int32_t tiles) { return c->s.S + (kTileWords * (size_t)tiles + 63) / 64 * 64; }

// Further copies of the bins of a segment of `ntiles` tiles where the layout has `tiles` and `have` copies already: one for
// sixteen tiles, seven at most, as long as S's memory has room for them behind the tables.
int32_t more_bins(const artopk_ctx* c, int32_t ntiles, int32_t tiles, int32_t have) {
  const int32_t want = std::min(ntiles / 16, 7);
  const int64_t words = ((int64_t)c->max_w * kMaxChunks + c->max_seg) * kHistBins;
  return kTileWords * (int64_t)tiles + 64 + (int64_t)(have + want) * kHistBins <= words ? want : 0;
}

// Whether a segmented selection goes by tiles (switches that were set hold for these, too).
bool segments_by_tiles(const artopk_ctx* c, const Plan& pl, int64_t n) {
  if (pl.tiles == 0 || c->stage_tiles == 0) return false;
  if (c->guess_min_n_set) return n >= c->guess_min_n;
  if (n < kSegTilesBareN)
    return !pl.some_bare && ((n >= kSegTilesMinN && pl.longest * 2 > n) ||
                             (n >= kSegTilesSomeN && pl.tiles >= kSegTilesEach * (int64_t)pl.nseg) ||
                             (n >= kSegTilesAllN && pl.tiles >= kSegTilesFew * (int64_t)pl.nseg));
  return pl.bare == 0 || pl.longest * pl.nseg > 4 * n || pl.nseg >= kSegTilesMany || pl.k_all * 5 > 2 * n ||
         (n >= kSegTilesFewBareN && pl.bare * 5 <= n);
}

// Descriptors for nseg > 1 segments; uploads them to the device table unless the
// same layout is already there, and makes the map of its tiles when they are first wanted
// (a launch that a program which changes between layouts would otherwise pay for on each of
// its calls: 4 M in 20 and in 27 segments in turn, two selections 139 us with it, 131 without).
// Copies from pageable memory, so the host buffer may be reused as soon as the call returns.
int segmented_plan(artopk_ctx* c, int64_t n, int32_t nseg, const int64_t* seg_off, const int64_t* seg_k,
                   const Plan** out) {
  const bool same = c->cached_n == n && (int32_t)c->cached_k.size() == nseg &&
                    memcmp(c->cached_off.data(), seg_off, sizeof(int64_t) * (nseg + 1)) == 0 &&
                    memcmp(c->cached_k.data(), seg_k, sizeof(int64_t) * nseg) == 0;
  if (!same) {
    Plan pl;
    pl.nseg = nseg;
    pl.use_table = true;
    pl.max_chunks = 1;
    pl.max_tiles = 1;
    pl.total_tiles = 0;
    pl.max_cap = 1;
    int64_t koff = 0, list_base = 0, flag_base = 0;
    int32_t chunk_begin = 0;
    for (int sgi = 0; sgi < nseg; ++sgi) {
      SegDesc d{};
      d.e_lo = seg_off[sgi];
      d.e_hi = seg_off[sgi + 1];
      const int64_t ns = d.e_hi - d.e_lo;
      int64_t mc = (int64_t)((double)kMaxChunks * (double)ns / (double)n);
      if (mc < 1) mc = 1;
      d.geom = make_geom(d.e_lo, d.e_hi, mc);
      d.koff = koff;
      d.list_base = list_base;
      d.flag_base = flag_base;
      d.chunk_begin = chunk_begin;
      d.k = (uint32_t)seg_k[sgi];
      d.cap = (uint32_t)seg_list_cap(ns, seg_k[sgi]);
      d.vec = -1;
      d.hreps = 1;
      d.tile_begin = pl.tiles;
      d.ntiles = (int32_t)((d.e_hi - d.e_lo / 32 * 32 + kMarkTile - 1) / kMarkTile);
      pl.tiles += d.ntiles;
      pl.longest = std::max(pl.longest, ns);
      if (ns > kShortBare && !SegSample(d.e_lo, d.e_hi, seg_k[sgi]).has_pieces(d.e_lo, d.e_hi, d.ntiles)) {
        pl.some_bare = true;
        if (ns > kMarkTile) pl.bare += ns;
      }
      if (d.e_lo % kPassTile != 0) pl.tiles_aligned = false;
      koff += seg_k[sgi];
      list_base += ((int64_t)d.cap + 3) / 4 * 4;
      const int64_t tiles = tiles_of_range(d.e_lo, d.e_hi);
      flag_base += tiles;
      chunk_begin += d.geom.nchunks;
      if (d.geom.nchunks > pl.max_chunks) pl.max_chunks = d.geom.nchunks;
      if (tiles > pl.max_tiles) pl.max_tiles = tiles;
      if ((int64_t)d.cap > pl.max_cap) pl.max_cap = d.cap;
      pl.desc.push_back(d);
    }
    pl.total_tiles = flag_base;
    pl.k_all = koff;
    if (list_base > c->s.list_entries || flag_base > c->s.max_tiles || chunk_begin > kMaxChunks + c->max_seg)
      return fail(c, ARTOPK_EINVAL, "segment layout exceeds the scratch sized at artopk_create");
    for (SegDesc& d : pl.desc) {
      d.group_begin = pl.tile_groups;
      pl.tile_groups += (d.ntiles + kTileWaves - 1) / kTileWaves;
      d.bins_begin = pl.more_bins;
      d.bins_more = more_bins(c, d.ntiles, pl.tiles, pl.more_bins);
      pl.more_bins += d.bins_more;
    }
    HIP_TRY(c, hipMemcpyAsync(c->s.table_dev, pl.desc.data(), sizeof(SegDesc) * nseg, hipMemcpyHostToDevice,
                              c->stream));
    // one block per chunk of the layout for the per-chunk kernels (a (chunks, segments) grid of a layout
    // with one long and many short segments is mostly blocks that find nothing to do)
    std::vector<uint32_t> cmap;
    cmap.reserve((size_t)chunk_begin);
    for (int sgi = 0; sgi < nseg; ++sgi)
      for (int32_t ch = 0; ch < pl.desc[sgi].geom.nchunks; ++ch) cmap.push_back(((uint32_t)sgi << 16) | (uint32_t)ch);
    HIP_TRY(c, hipMemcpyAsync(c->s.chunk_map, cmap.data(), sizeof(uint32_t) * cmap.size(), hipMemcpyHostToDevice,
                              c->stream));
    pl.total_chunks = chunk_begin;
    if ((int64_t)nseg * kPassTile > n || pl.tiles > c->s.map_tiles) pl.tiles = 0;
    c->cached_plan = pl;
    c->cached_map = false;
    c->cached_n = n;
    c->cached_off.assign(seg_off, seg_off + nseg + 1);
    c->cached_k.assign(seg_k, seg_k + nseg);
  }
  if (!c->cached_map && segments_by_tiles(c, c->cached_plan, n)) {
    hipLaunchKernelGGL(k_tile_map, dim3((unsigned)nseg), dim3(256), 0, c->stream, c->s.table_dev, c->s.tile_map,
                       reinterpret_cast<uint2*>(c->s.tile_map + c->s.map_tiles));
    HIP_TRY(c, hipGetLastError());
    // (a recorded launch has not run yet: the next call that goes by tiles makes the map again)
    hipStreamCaptureStatus capture = hipStreamCaptureStatusActive;
    if (hipStreamIsCapturing(c->stream, &capture) != hipSuccess) (void)hipGetLastError();
    c->cached_map = capture == hipStreamCaptureStatusNone;
  }
  *out = &c->cached_plan;
  return ARTOPK_OK;
}

SelParams make_params(const artopk_ctx* c, const Plan& pl, const PtrTable& tab, int64_t n, int32_t* idx_out,
                      float* vals_row, int slot_by_leader, bool hist_from_pass) {
  const Scratch& s = c->s;
  SelParams p;
  p.tab = tab;
  p.leader_dev = s.leader_dev;
  p.n = n;
  p.hcopies = s.h_all;
  p.hcopy_stride = kSlotWords;
  p.h_all = hist_from_pass ? s.h_all : nullptr;
  p.mask = nullptr;
  p.mask_stride = s.mask_stride;
  p.tiles = TileBuf{nullptr, nullptr, 0, 0, 0};
  p.use_mcount = 0;
  p.from_list = 0;
  p.after_mask = 0;
  p.only_if_need_full = 0;
  p.zero_base = s.zero_base;
  p.flags = s.flags;
  p.S = s.S;
  p.chunk_off = s.chunk_off;
  p.list = s.list;
  p.idx_out = idx_out;
  p.vals_row = vals_row;
  p.zero_vec = nullptr;
  p.err = s.err_dev;
  p.batch = pl.batch ? 1 : 0;
  const int64_t k_all = pl.batch ? pl.k_all * pl.nseg : pl.k_all;
  p.k_all = k_all < UINT32_MAX ? (uint32_t)k_all : UINT32_MAX;
  p.list_stride = pl.list_stride;
  p.flag_stride = pl.batch ? pl.max_tiles : 0;
  p.table = pl.use_table ? s.table_dev : nullptr;
  p.chunk_map = (pl.use_table && pl.total_chunks > 0) ? s.chunk_map : nullptr;
  p.slot_by_leader = slot_by_leader;
  p.one = pl.desc[0];
  return p;
}

// Clears the per-segment scratch blocks and the look-back flags of a plan, and the
// whole-vector histograms of the first hist_slots slots a fused pass is about to fill.
// leader >= 0 also records a host-known leader (and copies it to leader_out).
int enqueue_clear(artopk_ctx* c, const Plan& pl, int hist_slots, int32_t leader = -1,
                  int32_t* leader_out = nullptr, bool tiles = false) {
  Scratch& s = c->s;
  const size_t words1 = (size_t)pl.nseg * kSegWords;
  // (the selection by tiles has no look-back flags, but copies of bins)
  const size_t words2 = tiles ? (size_t)pl.more_bins * kHistBins : (size_t)pl.total_tiles * kNumLookback * 2;
  uint32_t* const range2 = tiles ? tile_more_bins(c, pl.tiles) : reinterpret_cast<uint32_t*>(s.flags);
  // (a plan with histograms of its own uses h_all's memory for their copies; no pass fills slots then)
  const size_t words3 = hist_slots > 0 ? (size_t)hist_slots * kSlotWords : pl.hist_words;
  const size_t total = words1 + words2 + words3;
  int blocks = (int)((total + 256 * 8 - 1) / (256 * 8));
  if (blocks < 1) blocks = 1;
  if (blocks > c->num_cu * 4) blocks = c->num_cu * 4;
  hipLaunchKernelGGL(k_fill_zero, dim3(blocks), dim3(256), 0, c->stream, s.zero_base, words1,
                     range2, words2, s.h_all, words3, leader,
                     leader >= 0 ? s.leader_dev : nullptr, leader_out);
  HIP_TRY(c, hipGetLastError());
  return ARTOPK_OK;
}

// Launches the fused pass over grid.y workers with the wanted options.
template <int STATS, int HIST, int GT>
void launch_pass_a_g(artopk_ctx* c, dim3 grid, const PtrTable& g, const PtrTable& r, int64_t n, const ChunkGeom& geom,
                     int hist_worker, bool by_tile) {
  Scratch& s = c->s;
  if (c->pass_a_nt)
    hipLaunchKernelGGL((k_pass_a<STATS, HIST, true, GT, kPassAThreads, kPassAU>), grid, dim3(kPassAThreads), 0,
                       c->stream, g, r, n, geom, hist_worker, by_tile ? nullptr : s.S, s.h_all, s.partials);
  else
    hipLaunchKernelGGL((k_pass_a<STATS, HIST, false, GT, kPassAThreads, kPassAU>), grid, dim3(kPassAThreads), 0,
                       c->stream, g, r, n, geom, hist_worker, by_tile ? nullptr : s.S, s.h_all, s.partials);
}

template <int STATS, int HIST>
void launch_pass_a_t(artopk_ctx* c, dim3 grid, const PtrTable& g, const PtrTable& r, int64_t n, const ChunkGeom& geom,
                     int hist_worker, bool by_tile) {
  if (c->g_type == ARTOPK_G_BF16)
    launch_pass_a_g<STATS, HIST, kGBF16>(c, grid, g, r, n, geom, hist_worker, by_tile);
  else if (c->g_type == ARTOPK_G_F16)
    launch_pass_a_g<STATS, HIST, kGF16>(c, grid, g, r, n, geom, hist_worker, by_tile);
  else
    launch_pass_a_g<STATS, HIST, kGF32>(c, grid, g, r, n, geom, hist_worker, by_tile);
}

void launch_pass_a(artopk_ctx* c, int stats, int hist, dim3 grid, const PtrTable& g, const PtrTable& r, int64_t n,
                   const ChunkGeom& geom, int hist_worker, bool by_tile = false) {
#define PASS_A_CASE(S_, H_) \
  if (stats == S_ && hist == H_) return launch_pass_a_t<S_, H_>(c, grid, g, r, n, geom, hist_worker, by_tile)
  PASS_A_CASE(0, 0);
  PASS_A_CASE(0, 1);
  PASS_A_CASE(0, 2);
  PASS_A_CASE(1, 0);
  PASS_A_CASE(1, 2);
  PASS_A_CASE(2, 0);
  PASS_A_CASE(2, 2);
#undef PASS_A_CASE
}

// Blocks per worker of a streaming pass that strides over the tiles of n elements.
int pass_blocks(int64_t n) {
  const int64_t ntiles = (n + kPassTile - 1) / kPassTile;
  return (int)(ntiles < kMaxPassBlocks ? ntiles : kMaxPassBlocks);
}

// The other workers' pass does best with fewer, longer-lived blocks (measured on 138 M x 3: 0.84 ms
// with 512 per worker against 0.85 - 0.87 with 1024 - 2048; no difference on 1e9 x 7), the marking
// pass with many (1e9 x 8: 16.35 ms with 4096 per worker, 16.55 with 2048).
int rest_blocks(int64_t n) {
  const int64_t ntiles = (n + kPassTile - 1) / kPassTile;
  return (int)(ntiles < 512 ? ntiles : 512);
}

// The fused pass of the guess route over the first nw workers of the tables (worker y in slot y).
template <int STATS, int GT>
void launch_pass_mark_g(artopk_ctx* c, int nw, const PtrTable& g, const PtrTable& r, int64_t n, int64_t chunk_elems) {
  Scratch& s = c->s;
  const dim3 grid(pass_blocks(n), nw);
  if (c->pass_a_nt)
    hipLaunchKernelGGL((k_pass_mark<STATS, true, GT, kPassAThreads, kPassAU>), grid, dim3(kPassAThreads), 0, c->stream, g, r,
                       n, chunk_elems, s.h_all, s.mask, s.mask_stride, s.partials);
  else
    hipLaunchKernelGGL((k_pass_mark<STATS, false, GT, kPassAThreads, kPassAU>), grid, dim3(kPassAThreads), 0, c->stream, g, r,
                       n, chunk_elems, s.h_all, s.mask, s.mask_stride, s.partials);
}

template <int STATS>
void launch_pass_mark_t(artopk_ctx* c, int nw, const PtrTable& g, const PtrTable& r, int64_t n, int64_t chunk_elems) {
  if (c->g_type == ARTOPK_G_BF16)
    launch_pass_mark_g<STATS, kGBF16>(c, nw, g, r, n, chunk_elems);
  else if (c->g_type == ARTOPK_G_F16)
    launch_pass_mark_g<STATS, kGF16>(c, nw, g, r, n, chunk_elems);
  else
    launch_pass_mark_g<STATS, kGF32>(c, nw, g, r, n, chunk_elems);
}

void launch_pass_mark(artopk_ctx* c, int stats, int nw, const PtrTable& g, const PtrTable& r, int64_t n,
                      int64_t chunk_elems) {
  if (stats == 0) return launch_pass_mark_t<0>(c, nw, g, r, n, chunk_elems);
  if (stats == 1) return launch_pass_mark_t<1>(c, nw, g, r, n, chunk_elems);
  return launch_pass_mark_t<2>(c, nw, g, r, n, chunk_elems);
}

// The striding pass without a bound: error-feedback add and statistics of all w workers (per-block
// moments of pass_blocks(n) blocks per worker in partials).
template <int STATS, int GT>
void launch_pass_plain_g(artopk_ctx* c, int nw, const PtrTable& g, const PtrTable& r, int64_t n) {
  Scratch& s = c->s;
  const dim3 grid(pass_blocks(n), nw);
  if (c->pass_a_nt)
    hipLaunchKernelGGL((k_pass_mark<STATS, true, GT, kPassAThreads, kPassAU, true>), grid, dim3(kPassAThreads), 0,
                       c->stream, g, r, n, (int64_t)kPassTile, s.h_all, s.mask, s.mask_stride, s.partials);
  else
    hipLaunchKernelGGL((k_pass_mark<STATS, false, GT, kPassAThreads, kPassAU, true>), grid, dim3(kPassAThreads), 0,
                       c->stream, g, r, n, (int64_t)kPassTile, s.h_all, s.mask, s.mask_stride, s.partials);
}

template <int STATS>
void launch_pass_plain_t(artopk_ctx* c, int nw, const PtrTable& g, const PtrTable& r, int64_t n) {
  if (c->g_type == ARTOPK_G_BF16)
    launch_pass_plain_g<STATS, kGBF16>(c, nw, g, r, n);
  else if (c->g_type == ARTOPK_G_F16)
    launch_pass_plain_g<STATS, kGF16>(c, nw, g, r, n);
  else
    launch_pass_plain_g<STATS, kGF32>(c, nw, g, r, n);
}

void launch_pass_plain(artopk_ctx* c, int stats, int nw, const PtrTable& g, const PtrTable& r, int64_t n) {
  if (stats == 0) return launch_pass_plain_t<0>(c, nw, g, r, n);
  if (stats == 1) return launch_pass_plain_t<1>(c, nw, g, r, n);
  return launch_pass_plain_t<2>(c, nw, g, r, n);
}

template <int GT>
void launch_pass_rest_g(artopk_ctx* c, dim3 grid, const PtrTable& g, const PtrTable& r, int w, int leader, int64_t n,
                        const int32_t* idx, int64_t k, float* vals) {
  Scratch& s = c->s;
  if (c->pass_a_nt)
    hipLaunchKernelGGL((k_pass_rest<true, GT, kPassRestThreads, kPassRestU>), grid, dim3(kPassRestThreads), 0, c->stream,
                       g, r, w, leader, n, idx, k, vals, s.tile_start, s.err_dev);
  else
    hipLaunchKernelGGL((k_pass_rest<false, GT, kPassRestThreads, kPassRestU>), grid, dim3(kPassRestThreads), 0, c->stream,
                       g, r, w, leader, n, idx, k, vals, s.tile_start, s.err_dev);
}

// The number of kept indices below every tile of the streaming passes.
void enqueue_tile_starts(artopk_ctx* c, const int32_t* idx, int64_t n, int64_t k) {
  const int32_t ntiles = (int32_t)((n + kPassTile - 1) / kPassTile);
  // many kept indices per tile: a search per tile boundary beats a thread per index
  // (138 M elements, one in ten kept: 20 us with a thread per index)
  if (k > (int64_t)1024 * ntiles)
    hipLaunchKernelGGL(k_tile_starts_search, dim3((unsigned)(ntiles / 256 + 1)), dim3(256), 0, c->stream, idx, k,
                       ntiles, c->s.tile_start);
  else
    hipLaunchKernelGGL(k_tile_starts, dim3((unsigned)((k + 255) / 256)), dim3(256), 0, c->stream, idx, k, ntiles,
                       c->s.tile_start);
}

// The other workers' streaming pass (leader known, idx final), striding over the tiles;
// k_tile_starts must have run on idx.
void launch_pass_rest(artopk_ctx* c, const PtrTable& g, const PtrTable& r, int w, int leader, int64_t n,
                      const int32_t* idx, int64_t k, float* vals) {
  const dim3 grid(rest_blocks(n), w - 1);
  if (c->g_type == ARTOPK_G_BF16)
    launch_pass_rest_g<kGBF16>(c, grid, g, r, w, leader, n, idx, k, vals);
  else if (c->g_type == ARTOPK_G_F16)
    launch_pass_rest_g<kGF16>(c, grid, g, r, w, leader, n, idx, k, vals);
  else
    launch_pass_rest_g<kGF32>(c, grid, g, r, w, leader, n, idx, k, vals);
}

// Whether a flat step on n elements keeping k uses the sampled threshold guess.
struct GuessPlan {
  bool on = false;
  int runs = 0;
  int64_t stride = 0;
  uint32_t m_hi = 0;
  uint32_t m_mid = 0, m_lo = 0;  // with tiles: the sample's share of k, and as far on the other side
  int32_t span = 0;      // elements per piece of the read-only marking pass
  uint32_t m_max = 0xffffffffu;  // more sample keys at or above a bound than this: no bound
  int32_t tile_cap = 0;  // entries per piece of it
  bool tiles = false;    // one vector whose marks are handed on by tiles
};

// known: the leader is known up front, and its pass alone will mark.  (Not so with a single worker whose leader comes from the
// data or the counter: such a step takes the mask, and with it the mask's lines: 25.6 M x 1, one in a hundred / in ten kept,
// histogram route 167/227 us, mask 181/286; 13 M x 1 104/135 and 119/172.)
GuessPlan plan_guess(const artopk_ctx* c, int64_t n, int64_t k, bool known) {
  GuessPlan gp;
  if (c->s.mask == nullptr || n < (known && !c->guess_min_n_set ? kTilesMinN : c->guess_min_n)) return gp;
  int64_t runs = n / (4 * kGuessRun);  // at most a quarter of the vector
  if (runs > 16384) runs = 16384;
  if (runs < 256) return gp;
  const double sample = (double)(runs * kGuessRun);
  // keys of the sample expected above the true threshold, plus six standard deviations and a few
  const double expect = (double)k * sample / (double)n;
  const double margin = 6.0 * std::sqrt(expect) + 8.0;
  gp.runs = (int)runs;
  gp.stride = n / runs;
  gp.m_hi = (uint32_t)std::ceil(expect + margin);
  gp.m_mid = (uint32_t)std::max(1.0, expect + 0.5);
  gp.m_lo = (uint32_t)std::max(1.0, expect - margin);
  // A leader known up front hands its marks on by tiles (k_mark_tiles), unless the option forbids it or a tile's piece
  // would not hold its share of what reaches the bound, and six standard deviations: up to one in seven kept (histogram
  // route / tiles, us a step, one in eight 12.6 M x 2 167/162, 25.6 M x 2 270/239, 138 M x 2 1358/948, x 4 1980/1585, one in
  // seven 171/166, 280/250, 1425/1027, 2051/1654).  Very sparse selections on very long vectors do without, as the mask then is
  // the smaller thing to write (histogram route / mask / tiles, us a step: 138 M x 4, one in 3000 kept 1386/1266/1269, in
  // 1000 1396/1282/1264, in 250 1419/1321/1269, in 100 1468/1413/1294; mask / tiles, x 2, one in 3000, 1000, 700, 500 and 250,
  // 180 M 923/934 934/937 939/944 949/947 991/948, 220 M 1117/1144 1140/1144 1148/1150 1152/1156 1216/1159, 268 M 1362/1387
  // 1355/1389 1368/1399 1379/1400 1464/1403, 300 M 1518/1557 1530/1554 1536/1553 1553/1562 1657/1571; 25.6 M x 4, one in 1000
  // 306/280, in 100 323/290; below kTilesMinN see there).
  const double per_tile = (double)gp.m_hi / sample * (double)kMarkTile;
  const bool worth = c->stage_tiles == 2 || n < ((int64_t)5 << 25) || k * 500 >= n;
  gp.tiles = c->stage_tiles != 0 && known && worth && per_tile + 6.0 * std::sqrt(per_tile) <= (double)kMarkMax;
  // A selection of more than one element in 32 is not worth fetching entry by entry from the mask; nor is the mask on
  // vectors that the tiles alone would take.
  if (!gp.tiles && (k * 32 > n || n < c->guess_min_n)) return gp;
  gp.on = (int64_t)gp.m_hi <= runs * kGuessRun;
  gp.tiles = gp.tiles && gp.on;
  return gp;
}

// The guess of a selection on `vectors` vectors as they are (no pass writes them): a smaller sample, since a
// longer list costs little here (nothing has to be given back from it), and pieces wherever they fit.
GuessPlan plan_guess_read(const artopk_ctx* c, int64_t n, int64_t k, int vectors, int64_t list_cap) {
  GuessPlan gp;
  if (c->s.mask == nullptr || (c->guess_min_n_set ? n < c->guess_min_n : n * vectors < kReadGuessMinN)) return gp;
  if (k * 32 > n) return gp;
  int64_t runs = n / (4 * kGuessRun);
  if (runs > 4096) runs = 4096;
  if (runs < 256) return gp;
  gp.runs = (int)runs;
  gp.stride = n / runs;
  const double sample = (double)(runs * kGuessRun);
  const double expect = (double)k * sample / (double)n;
  gp.m_hi = (uint32_t)std::ceil(expect + 6.0 * std::sqrt(expect) + 8.0);
  if ((double)gp.m_hi > sample) return gp;
  // what k_pick_mask accepts: at most k + n/8 keys, and no more than the list takes
  int64_t limit = k + (n >> 3);
  if (limit > list_cap) limit = list_cap;
  gp.m_max = (uint32_t)((double)limit * sample / (double)n);
  if (gp.m_max <= gp.m_hi) return gp;
  // entries a span hands on: the bound is the lower edge of a top-digit bin (up to about 15 % more keys than
  // the sample's m_hi-th largest), plus four standard deviations of a span's count (a span with more is marked
  // a second time)
  gp.span = n * vectors < ((int64_t)1 << 23) ? kSpanStep : 4 * kSpanStep;  // (short vectors need the spans to fill the chip)
  const double per_span = 1.15 * (double)gp.m_hi / sample * (double)gp.span;
  const int64_t want = ((int64_t)std::ceil(per_span + 4.0 * std::sqrt(per_span) + 8.0) + 15) / 16 * 16;
  const int64_t nspans = (n + gp.span - 1) / gp.span;
  if (nspans * want * vectors > c->s.tilebuf_entries) return gp;
  gp.tile_cap = (int32_t)want;
  // A bound that more keys reach than the pieces hold on average (many values equal, or in one top digit, just below
  // the threshold) has nearly every span marked twice.  From kTwiceMaxN elements on it counts as none: the histogram
  // route is then the better one (one in a hundred kept, us, marked twice / no bound: one in twenty equal just below,
  // 1 x 32 M 129/142, 40 M 156/158, 50 M 175/170, 138 M 390/359, 400 M 1002/887, 8 x 4 M 155/140, 4 x 12 M 185/172;
  // uniform values, 1 x 32 M 112/130, 40 M 127/138, 50 M 143/156, 60 M 172/173, 400 M 834/803, 2 x 20 M 142/145, 4 x 12 M
  // 160/152).
  const double held = sample * (double)want / (double)gp.span;
  if (n * vectors >= kTwiceMaxN && held < (double)gp.m_max) gp.m_max = (uint32_t)held;
  gp.on = true;
  return gp;
}

// The spans' pieces of the marking pass on vectors that are only read (slots 0, 1, ...); their counts lie in
// the memory of the vectors' masks, which this route does not use.
TileBuf span_buf(const artopk_ctx* c, const GuessPlan& gp, int64_t n) {
  const int64_t nspans = (n + gp.span - 1) / gp.span;
  return TileBuf{c->s.tilebuf, reinterpret_cast<uint32_t*>(c->s.mask), nspans * gp.tile_cap, 2 * c->s.mask_stride,
                 gp.tile_cap, gp.span};
}

// The marking pass over the first nv vectors of the table.
void launch_mark_spans(artopk_ctx* c, const GuessPlan& gp, int nv, const PtrTable& x, int64_t n, int64_t chunk_elems) {
  const int64_t nspans = (n + gp.span - 1) / gp.span;
  int64_t blocks = (nspans + 3) / 4;
  if (blocks > (int64_t)c->num_cu * 8) blocks = (int64_t)c->num_cu * 8;
  const dim3 grid((unsigned)blocks, (unsigned)nv);
  const TileBuf tb = span_buf(c, gp, n);
  if (c->pass_a_nt)
    hipLaunchKernelGGL(k_mark_spans<true>, grid, dim3(256), 0, c->stream, x, n, chunk_elems, c->s.h_all, tb);
  else
    hipLaunchKernelGGL(k_mark_spans<false>, grid, dim3(256), 0, c->stream, x, n, chunk_elems, c->s.h_all, tb);
}

// The leader's pass of a segmented step: one block per chunk of the layout, which also builds the histograms
// that enqueue_select would otherwise read the vector for.
template <int GT>
void launch_pass_seg(artopk_ctx* c, const Plan& pl, const PtrTable& r, int64_t n, const float* g, float* res) {
  const SelParams p = make_params(c, pl, r, n, nullptr, nullptr, 0, false);
  if (c->pass_a_nt)
    hipLaunchKernelGGL((k_pass_seg<true, GT, 1024>), dim3((unsigned)pl.total_chunks), dim3(1024), 0, c->stream, p, g, res);
  else
    hipLaunchKernelGGL((k_pass_seg<false, GT, 1024>), dim3((unsigned)pl.total_chunks), dim3(1024), 0, c->stream, p, g, res);
}

// Samples the first nvec vectors of (g + residual) into slots 0 .. nvec-1 (cleared beforehand).
void enqueue_guess(artopk_ctx* c, const GuessPlan& gp, const PtrTable& g, const PtrTable& res, int nvec,
                   bool read_only = false) {
  // about 128 blocks over all vectors (measured: 8 vectors take 70 us with 64 blocks each, 32 us
  // with 16; one vector 15 us with 64 blocks, 19 us with 16)
  int gblocks = 128 / nvec;
  if (gblocks > 64) gblocks = 64;
  if (gblocks < 8) gblocks = 8;
  if (read_only) gblocks = (gp.runs + 255) / 256;  // one run a thread
#define GUESS_LAUNCH(GT_) \
  hipLaunchKernelGGL(k_guess<GT_>, dim3(gblocks, nvec), dim3(256), 0, c->stream, g, res, c->s.h_all, gp.runs, gp.stride, \
                     gp.m_hi, gp.m_max)
  if (read_only)
    GUESS_LAUNCH(kGNone);
  else if (c->g_type == ARTOPK_G_BF16)
    GUESS_LAUNCH(kGBF16);
  else if (c->g_type == ARTOPK_G_F16)
    GUESS_LAUNCH(kGF16);
  else
    GUESS_LAUNCH(kGF32);
#undef GUESS_LAUNCH
}

// How k_tail takes a selection: ranges (blocks) a vector, and rows of 256 elements in each of a wave's pieces (log2).
struct TailPlan {
  int32_t ranges = 0;  // 0: the list kernels are the better way
  int32_t row_log2 = 0;
};

TailPlan tail_plan(const Plan& pl, int64_t n, int source) {
  TailPlan t;
  if (pl.use_table || pl.nseg > kTailRanges || pl.lists) return t;
  const int64_t waves = (int64_t)(kTailRanges / pl.nseg) * kTailWaves;
  const int64_t elems = ((n + waves - 1) / waves + kTailRow - 1) / kTailRow * kTailRow;
  // Survivors a wave is expected to have: the candidates below the threshold, or the guess' margin and the rest of its
  // bin, come to less than half of k.
  if (1.5 * (double)pl.desc[0].k / (double)waves > (double)kTailKeep) return t;
  // (Denser ones, 138 M and one in 33: the list kernels read their entries from memory a few times less.)
  // With nothing there yet, two passes over the vector and short chunks stand up better to runs of large values, unless a
  // wave can keep all its elements (us, list kernels / this, normal values and a run: 8 x 2 M 100/66 98/123, 1 x 11.7 M
  // 61/58 66/92, 1 x 3 M 46/45 47/47, 16 x 1.2 M 98/72 94/117).
  if (source == kTailNone && (pl.nseg < 2 || elems > kTailKeep)) return t;
  // Behind a pass' counts the list kernels are measured against it up to 12.5 M elements (see k_tail; in one piece a wave,
  // longer vectors lost on layers and runs, 25.6 M x 4, list kernels / that: 358/334 normal values, 340/356, 370/444).
  if (source == kTailHist && elems > 6144) return t;
  // Up to 16 pieces a wave, and more where fewer blocks share a vector: every block reads what the others keep of theirs.
  const int32_t most = std::min(kTailPieces, 4096 / (kTailRanges / pl.nseg));
  while (((int64_t)kTailRow << t.row_log2) * most < elems) ++t.row_log2;
  t.ranges = (int32_t)std::min<int64_t>(kTailRanges / pl.nseg, (n + kTailWaves * kTailRow - 1) / (kTailWaves * kTailRow));
  return t;
}

// Top-k of every segment of the plan on the vector tab.p[*leader_dev]; the
// scratch must have been cleared.  If hist_ready the per-chunk suffix
// histograms are already in S (flat plans only: pass A built them, in slot
// *leader_dev if slot_by_leader, else in slot 0).  vals_row, if given, receives
// the leader's values at the selected indices.
int enqueue_select(artopk_ctx* c, const Plan& pl, const PtrTable& tab, int64_t n, int32_t* idx_out,
                   bool hist_ready, int slot_by_leader, float* vals_row = nullptr,
                   const LeaderArgs* leader_args = nullptr, bool guessed = false, float* zero_vec = nullptr,
                   int32_t first_slot = 0, const GuessPlan* spans = nullptr,
                   bool seg_hist_ready = false) {
  hipStream_t st = c->stream;
  const unsigned nseg = (unsigned)pl.nseg;
  SelParams p = make_params(c, pl, tab, n, idx_out, vals_row, (hist_ready || pl.batch) ? slot_by_leader : 0,
                            hist_ready);
  if (hist_ready) p.h_all += (size_t)first_slot * kSlotWords;  // (slots of a later group of a batch)
  p.S += (size_t)first_slot * kMaxChunks * kHistBins;
  p.zero_vec = zero_vec;
  LeaderArgs la{};
  if (leader_args) la = *leader_args;
  const int source = spans ? kTailSpans : hist_ready ? kTailHist : kTailNone;
  // (the leader's own selection in front of the other workers' pass gains 2 % of a step, and loses a third on a run)
  const TailPlan tp = (guessed && !spans) || zero_vec ? TailPlan{} : tail_plan(pl, n, source);
  c->last_one_launch = tp.ranges > 0 ? 1 : 0;
  c->last_tiles = 0;
  if (tp.ranges > 0) {
    if (spans) {
      p.tiles = span_buf(c, *spans, n);
      p.use_mcount = 1;
    }
    const dim3 grid((unsigned)tp.ranges, nseg), block(64 * kTailWaves);
    if (source == kTailSpans)
      hipLaunchKernelGGL(k_tail<kTailSpans>, grid, block, 0, st, p, la, tp.row_log2);
    else if (source == kTailHist)
      hipLaunchKernelGGL(k_tail<kTailHist>, grid, block, 0, st, p, la, tp.row_log2);
    else
      hipLaunchKernelGGL(k_tail<kTailNone>, grid, block, 0, st, p, la, tp.row_log2);
    HIP_TRY(c, hipGetLastError());
    return ARTOPK_OK;
  }
  // the per-chunk kernels: one block per chunk of a segmented layout, else a (chunks, segments) grid
  const dim3 chunk_grid = p.chunk_map ? dim3((unsigned)pl.total_chunks, 1) : dim3(pl.max_chunks, nseg);

  if (guessed && hist_ready) {
    // The fused pass marked and counted the keys reaching a guessed bound.  If the bound works out
    // the list is written from the mask and the threshold digit taken from the list; otherwise the
    // state says need_full, and the same two launches build the histogram of every key and pick
    // from that, after which the selection goes on as without a guess.
    p.mask = spans ? nullptr : c->s.mask + (size_t)first_slot * (size_t)c->s.mask_stride;
    if (spans) p.tiles = span_buf(c, *spans, n);
    p.use_mcount = 1;
    hipLaunchKernelGGL(k_pick_mask, dim3(1, nseg), dim3(1024), 0, st, p, la);
    SelParams pf = p;
    pf.h_all = nullptr;
    pf.only_if_need_full = 1;
    if (spans)
      hipLaunchKernelGGL(k_spans_or_hist, dim3(pl.max_chunks, nseg), dim3(1024), 0, st, p, pf);
    else
      hipLaunchKernelGGL((k_mask_or_hist<4>), dim3(pl.max_chunks, nseg), dim3(1024), 0, st, p, pf);
    SelParams pa = p;
    pa.after_mask = 1;
    hipLaunchKernelGGL(k_pick0, dim3(1, nseg), dim3(1024), 0, st, pa, LeaderArgs{});
  } else {
    if (!hist_ready && !seg_hist_ready) hipLaunchKernelGGL(k_hist0<1024>, chunk_grid, dim3(1024), 0, st, p);
    hipLaunchKernelGGL(k_pick0, dim3(1, nseg), dim3(1024), 0, st, p, la);
  }

  // The remaining kernels take tiles from a counter (or stride over the list), so any grid works:
  // about two blocks per compute unit over all segments together.
  const int64_t per_seg = ((int64_t)c->num_cu * 2 + nseg - 1) / nseg;
  // deeper array passes: they run only for segments whose level-1 survivors did not fit the list,
  // which cannot happen if the list takes the whole range
  const bool one_range = nseg == 1 || pl.batch;
  const bool always_fits = one_range && (int64_t)pl.desc[0].cap >= pl.desc[0].e_hi - pl.desc[0].e_lo;
  int cblocks = (int)(pl.max_tiles < per_seg ? pl.max_tiles : per_seg);
  if (cblocks < 1) cblocks = 1;

  int64_t lblocks = (pl.max_cap + 256 * 16 - 1) / (256 * 16);
  if (lblocks > per_seg * 2) lblocks = per_seg * 2;
  if (lblocks < 1) lblocks = 1;
  // level 1: ordered compaction of the array (4 waves, 16 consecutive elements per lane: best of the
  // shapes measured on the 138 M and 1 G workloads); on the guess route the same launch counts
  // the second digit over a list that was written from the mask
  const bool long_list = one_range && (int64_t)pl.desc[0].k * 32 > n;
  if (guessed && hist_ready) {
    const int64_t b1 = lblocks > pl.max_chunks ? lblocks : pl.max_chunks;
    if (spans)  // (half as many chunks as behind a fused pass)
      hipLaunchKernelGGL(k_level1<8>, dim3((unsigned)b1, nseg), dim3(512), 0, st, p);
    else
      hipLaunchKernelGGL(k_level1<kC1Waves>, dim3((unsigned)b1, nseg), dim3(64 * kC1Waves), 0, st, p);
  } else {
    // (8 waves a block: 21.6 against 27.6 us with 4 on 11.7 M elements, 35 against 38 us on 25.6 M in 54 segments)
    hipLaunchKernelGGL((k_compact1<8, kC1R>), chunk_grid, dim3(512), 0, st, p);
  }
  // A list of many millions of entries (one element in 32 kept, or more) is counted faster by the
  // lean kernel of its own (99 vs 66 us on 15 M entries: the merged one carries the array pass'
  // registers), which is worth the launch of an array pass that has nothing to do.
  if (always_fits) {
    hipLaunchKernelGGL(k_list_hist, dim3((unsigned)lblocks, nseg), dim3(256), 0, st, p, 2);
  } else if (long_list) {
    hipLaunchKernelGGL(k_compact, dim3(cblocks, nseg), dim3(kCompactThreads), 0, st, p);
    hipLaunchKernelGGL(k_list_hist, dim3((unsigned)lblocks, nseg), dim3(256), 0, st, p, 2);
  } else {  // the same launch is the level-2 array pass where the level-1 survivors did not fit the list
    const int64_t b2 = lblocks > cblocks ? lblocks : cblocks;
    hipLaunchKernelGGL(k_level2, dim3((unsigned)b2, nseg), dim3(kCompactThreads), 0, st, p);
  }
  int64_t ltiles = (pl.max_cap + kListTile - 1) / kListTile;
  int fblocks = (int)(ltiles < per_seg ? ltiles : per_seg);
  if (fblocks < 1) fblocks = 1;
  // (the same launch is the level-3 array pass where no list could be written)
  if (!always_fits && fblocks < cblocks) fblocks = cblocks;
  if (always_fits)
    hipLaunchKernelGGL(k_final<true>, dim3(fblocks, nseg), dim3(kCompactThreads), 0, st, p);
  else
    hipLaunchKernelGGL(k_final<false>, dim3(fblocks, nseg), dim3(kCompactThreads), 0, st, p);
  HIP_TRY(c, hipGetLastError());
  return ARTOPK_OK;
}

// A vector that is only read by tiles comes through the caches up to this length: the next selection on it may find it there
// (ordinary / non-temporal loads, us, one in a hundred, 54 segments: 25.6 M 81/81, 40 M 92/96, 60 M 107/112, 67 M 117/120,
// 80 M 134/130, 100 M 156/150, 138 M 198/187).  A step is the same either way (variance rule, x 8, 25.6 M 602/597, 60 M
// 1302/1292, 67 M 1436/1430, 80 M 1704/1702).
constexpr int64_t kCachedMaxN = (int64_t)1 << 26;

// The bounds and the marking.
template <int GT>
void launch_tiles(artopk_ctx* c, const SelParams& p, const TileArgs& a, const Plan& pl, const GuessPlan& gp, const float* g, float* res) {
  const dim3 block(kMarkThreads), mark_grid((unsigned)std::min<int32_t>(a.ntiles, 2 * kMaxPassBlocks));
  if (pl.use_table) {
    PtrTable gt{};
    gt.p[0] = const_cast<float*>(g);
    hipLaunchKernelGGL(k_guess_segs<GT>, dim3((unsigned)pl.nseg), dim3(1024), 0, c->stream, p, gt);
  } else if constexpr (GT != kGNone) {
    hipLaunchKernelGGL(k_guess_tiles<GT>, dim3((unsigned)((gp.runs + kGuessThreads - 1) / kGuessThreads)), dim3(kGuessThreads), 0, c->stream, g, res,
                       c->s.h_all, gp.runs, gp.stride, gp.m_hi, gp.m_mid, gp.m_lo, c->s.zero_base + kTileInfo);
  }
  if (c->pass_a_nt && (GT != kGNone || p.n > kCachedMaxN))
    hipLaunchKernelGGL((k_mark_tiles<true, GT>), mark_grid, block, 0, c->stream, p, a, g, res);
  else
    hipLaunchKernelGGL((k_mark_tiles<false, GT>), mark_grid, block, 0, c->stream, p, a, g, res);
}

template <bool APART>
void launch_tiles_rest(artopk_ctx* c, const SelParams& p, const TileArgs& a) {
  const dim3 groups((unsigned)a.ngroups), block(64 * kTileWaves);
  hipLaunchKernelGGL((k_tiles_digit<1, APART>), groups, block, 0, c->stream, p, a);
  hipLaunchKernelGGL((k_tiles_digit<2, APART>), groups, block, 0, c->stream, p, a);
  hipLaunchKernelGGL(k_tiles_count<APART>, groups, block, 0, c->stream, p, a);
  hipLaunchKernelGGL(k_tiles_out<APART>, groups, block, 0, c->stream, p, a);
}

// Selection by tiles (see TileArgs) on the leader's vector, leader_dev's, of tab, from the sample on; the scratch has been
// cleared.  g and res: its gradients, and itself, to be added up on the way, or nullptr.  zero: its kept entries become +0.0.
int enqueue_tiles(artopk_ctx* c, const Plan& pl, const PtrTable& tab, int64_t n, int32_t* idx_out, float* vals_row,
                  const GuessPlan& gp, const float* g, float* res, bool zero) {
  Scratch& s = c->s;
  c->last_one_launch = 0;
  c->last_tiles = pl.nseg;
  SelParams p = make_params(c, pl, tab, n, idx_out, vals_row, 0, false);
  p.zero_vec = zero ? res : nullptr;
  TileArgs a{};
  a.ntiles = pl.use_table ? pl.tiles : pl.desc[0].ntiles;
  a.ngroups = pl.use_table ? pl.tile_groups : (a.ntiles + kTileWaves - 1) / kTileWaves;
  a.map = pl.use_table ? s.tile_map : nullptr;
  a.groups = pl.use_table ? reinterpret_cast<const uint2*>(s.tile_map + s.map_tiles) : nullptr;
  a.pieces = s.tilebuf;
  // (nobody else has anything in S's memory now)
  a.kept = reinterpret_cast<uint64_t*>(s.S);
  a.held = s.S + kTileHeldAt * (size_t)a.ntiles;
  a.marked = s.S + kTileMarkedAt * (size_t)a.ntiles;
  a.above = s.S + kTileAboveAt * (size_t)a.ntiles;
  a.among = s.S + kTileAmongAt * (size_t)a.ntiles;
  a.slots = s.S + kTileSlotsAt * (size_t)a.ntiles;
  a.bins = pl.use_table ? s.zero_base + kSegHtop : s.h_all;
  a.bins_stride = pl.use_table ? kSegWords : 0;
  a.more_bins = pl.use_table ? tile_more_bins(c, a.ntiles) : s.h_all + kHistBins;
  a.any_full = s.zero_base + kTileInfo + kTileFull;
  a.tile_start = !pl.use_table || pl.tiles_aligned ? s.tile_start : nullptr;
  if (g == nullptr)
    launch_tiles<kGNone>(c, p, a, pl, gp, g, res);
  else if (c->g_type == ARTOPK_G_BF16)
    launch_tiles<kGBF16>(c, p, a, pl, gp, g, res);
  else if (c->g_type == ARTOPK_G_F16)
    launch_tiles<kGF16>(c, p, a, pl, gp, g, res);
  else
    launch_tiles<kGF32>(c, p, a, pl, gp, g, res);
  if (g != nullptr) prof_mark(c, 1);
  hipLaunchKernelGGL(k_tiles_pick, dim3((unsigned)pl.nseg), dim3(1024), 0, c->stream, p, a);
  hipLaunchKernelGGL(k_tiles_full, dim3((unsigned)std::min<int32_t>(a.ntiles, 2 * c->num_cu)), dim3(kMarkThreads), 0, c->stream, p, a);
  if (a.ntiles <= kTilesApart)
    launch_tiles_rest<true>(c, p, a);
  else
    launch_tiles_rest<false>(c, p, a);
  HIP_TRY(c, hipGetLastError());
  return ARTOPK_OK;
}

int enqueue_gather(artopk_ctx* c, const PtrTable& tab, int32_t w, int64_t n, const int32_t* idx, int64_t k,
                   float* vals, float* sum, bool zero) {
  const int blocks = (int)((k + 255) / 256);
  if (zero)
    hipLaunchKernelGGL(k_gather<true>, dim3(blocks), dim3(256), 0, c->stream, tab, (int)w, n, idx, k, vals, sum,
                       c->s.err_dev);
  else
    hipLaunchKernelGGL(k_gather<false>, dim3(blocks), dim3(256), 0, c->stream, tab, (int)w, n, idx, k, vals, sum,
                       c->s.err_dev);
  HIP_TRY(c, hipGetLastError());
  return ARTOPK_OK;
}

// tiles_ready: k_tile_starts has already run on this idx.
int enqueue_update_fill(artopk_ctx* c, float* update, int64_t n, const int32_t* idx, const float* sum,
                        int64_t k, bool tiles_ready = false) {
  // long vectors with few kept entries: zeros streamed tile by tile, values stored behind them
  // (measured on 138 M elements: faster at k = N / 1000, even at N / 100, 40 % slower at N / 10)
  if (n >= c->update_tiles_min_n && k * 128 <= n) {
    if (!tiles_ready) enqueue_tile_starts(c, idx, n, k);
    if (n < ((int64_t)1 << 28))  // (which kind of store the zeros take: measured, see the kernel)
      hipLaunchKernelGGL((k_update_tiles<kPassRestThreads, kPassRestU, true>), dim3(pass_blocks(n)),
                         dim3(kPassRestThreads), 0, c->stream, update, n, idx, sum, k, c->s.tile_start, c->s.err_dev);
    else
      hipLaunchKernelGGL((k_update_tiles<kPassRestThreads, kPassRestU, false>), dim3(pass_blocks(n)),
                         dim3(kPassRestThreads), 0, c->stream, update, n, idx, sum, k, c->s.tile_start, c->s.err_dev);
    HIP_TRY(c, hipGetLastError());
    return ARTOPK_OK;
  }
  const int64_t nchunk = (n + kFillChunk - 1) / kFillChunk;
  int blocks = (int)(nchunk < (int64_t)c->num_cu * 4 ? nchunk : (int64_t)c->num_cu * 4);
  if (blocks < 1) blocks = 1;
  // kept entries expected per 8192-element chunk decide how many are fetched per round
  const double per_chunk = (double)k / (double)n * kFillChunk;
  if (tiles_ready && n >= c->update_tiles_min_n) {
    // the tiles' first indices are there already: blocks stride over the tiles
    const int64_t ntiles = (n + kPassTile - 1) / kPassTile;
    const int tb = (int)(ntiles < (int64_t)c->num_cu * 4 ? ntiles : (int64_t)c->num_cu * 4);
    if (per_chunk <= 160.0)
      hipLaunchKernelGGL((k_update_fill_tiled<1>), dim3(tb), dim3(256), 0, c->stream, update, n, idx, sum, k, c->s.tile_start);
    else if (per_chunk <= 400.0)
      hipLaunchKernelGGL((k_update_fill_tiled<2>), dim3(tb), dim3(256), 0, c->stream, update, n, idx, sum, k, c->s.tile_start);
    else
      hipLaunchKernelGGL((k_update_fill_tiled<4>), dim3(tb), dim3(256), 0, c->stream, update, n, idx, sum, k, c->s.tile_start);
    HIP_TRY(c, hipGetLastError());
    return ARTOPK_OK;
  }
  if (per_chunk <= 160.0) {
    hipLaunchKernelGGL((k_update_fill<1>), dim3(blocks), dim3(256), 0, c->stream, update, n, idx, sum, k);
  } else if (per_chunk <= 400.0) {
    hipLaunchKernelGGL((k_update_fill<2>), dim3(blocks), dim3(256), 0, c->stream, update, n, idx, sum, k);
  } else {
    hipLaunchKernelGGL((k_update_fill<4>), dim3(blocks), dim3(256), 0, c->stream, update, n, idx, sum, k);
  }
  HIP_TRY(c, hipGetLastError());
  return ARTOPK_OK;
}


// Top-k of each of w whole vectors (row r of idx_rows, and of val_rows if given), several at a time in one
// launch set (8 x 25.6 M on the histogram route: 768 us one after the other, 438 together).  A context's list is sized for one selection, so a batch shares it out: as many vectors at a
// time as leave each room for 1.25 k + n/128 entries (what a list usually holds, with some ties).
//   hist_ready: the fused pass has left vector r's histograms (or, if guessed, its mask) in slot r.
//   Otherwise a sampled bound and a read-only marking pass (k_mark_spans) take the place of the
//   two passes over the vector, histograms and compaction, that the histogram route needs.
int enqueue_topk_rows(artopk_ctx* c, const PtrTable& tab, int32_t w, int64_t n, int64_t k, int32_t* idx_rows,
                      float* val_rows, bool hist_ready, bool guessed) {
  Scratch& s = c->s;
  const int64_t room = s.list_entries - kCompactTile;  // (the final pass reads up to a tile behind a list's end)
  int64_t need = k + k / 4 + (n / 128 > 4096 ? n / 128 : 4096);
  if (need > n) need = n;
  auto group_size = [&](int64_t most) {
    if (most > w) most = w;
    if (most > kMaxBatch) most = kMaxBatch;
    if (most < 1) most = 1;
    const int64_t groups = (w + most - 1) / most;
    return (int32_t)((w + groups - 1) / groups);
  };
  int32_t per = group_size(room / ((need + 3) / 4 * 4));
  auto cap_of = [&](int32_t vectors) {
    const int64_t stride = vectors == 1 ? room : room / vectors / 4 * 4;
    return stride < n ? stride : n;
  };
  GuessPlan gp;
  if (!hist_ready) {
    gp = plan_guess_read(c, n, k, per, vec_cap(c, cap_of(per)));
    for (int32_t fewer = per - 1; !gp.on && fewer >= 1; --fewer) {  // fewer at a time may leave room for the pieces
      gp = plan_guess_read(c, n, k, fewer, vec_cap(c, cap_of(fewer)));
      if (gp.on) {
        per = group_size(fewer);
        gp = plan_guess_read(c, n, k, per, vec_cap(c, cap_of(per)));
      }
    }
  }
  const bool marks = guessed || gp.on;
  c->last_guessed = marks ? 1 : 0;
  for (int32_t r0 = 0; r0 < w; r0 += per) {
    const int32_t nv = w - r0 < per ? w - r0 : per;
    // The fused pass counted per chunk of its own layout; the two passes of the histogram route do best with about
    // two thousand chunks over all vectors.  Behind the read-only marking one block copies a chunk's pieces, two
    // blocks fit a compute unit, and each is mostly latency: one round of 512 blocks up to 2e8 elements, two beyond
    // (us, one in a hundred kept, 512 / 1024 / 2048 chunks: 1 x 25.6 M 78/85/85, 60 M 109/115, 138 M 180/183/183, 200 M
    // 243/247, 230 M 275/275, 270 M 318/317, 330 M 367/369, 400 M 492/477/477; 4 x 40 M 218/219, 60 M 288/296; 8 x 20 M
    // 219/221, 25.6 M 271/266/274, 30 M 340/346; 256 chunks: 25.6 M 76, 138 M 183, 400 M 492).
    int64_t max_chunks = kMaxChunks;
    if (gp.on)
      max_chunks = (n * nv <= ((int64_t)3 << 26) ? kMaxChunks / 2 : kMaxChunks) / nv;
    else if (!hist_ready && nv > 1)
      max_chunks = 2 * kMaxChunks / nv;
    if (max_chunks < 64) max_chunks = 64;
    if (max_chunks > kMaxChunks) max_chunks = kMaxChunks;
    Plan pl = flat_plan(c, n, k, -1, marks, !hist_ready && !gp.on, max_chunks);
    pl.nseg = nv;
    pl.batch = true;
    pl.list_stride = nv == 1 ? 0 : room / nv / 4 * 4;
    pl.desc[0].cap = (uint32_t)vec_cap(c, cap_of(nv));
    pl.max_cap = pl.desc[0].cap;
    pl.total_tiles = pl.max_tiles * nv;
    if (pl.hist_words) pl.hist_words = (size_t)nv * kSlotWords;
    int rc = enqueue_clear(c, pl, gp.on ? nv : 0);
    if (rc) return rc;
    PtrTable t;
    for (int i = 0; i < kMaxW; ++i) t.p[i] = i < nv ? tab.p[r0 + i] : nullptr;
    if (gp.on) {
      enqueue_guess(c, gp, t, t, nv, true);
      launch_mark_spans(c, gp, nv, t, n, pl.desc[0].geom.chunk_elems);
    }
    if ((rc = enqueue_select(c, pl, t, n, idx_rows + (size_t)r0 * (size_t)k, hist_ready || gp.on, 1,
                             val_rows ? val_rows + (size_t)r0 * (size_t)k : nullptr, nullptr, marks, nullptr,
                             hist_ready ? r0 : 0, gp.on ? &gp : nullptr)))
      return rc;
  }
  return ARTOPK_OK;
}

// Every worker's own Top-k (indices ascending, values) and the squared norm of its k values;
// argmax (first maximum) goes to leader_dev and, if given, argmax_out.  With hist_ready the
// per-chunk histograms of all workers are already in S (pass A with histograms for every worker).
int enqueue_topk_workers(artopk_ctx* c, const PtrTable& tab, int32_t w, int64_t n, int64_t k, int32_t* idx_rows,
                         float* val_rows, double* sqnorm_out, int32_t* argmax_out, bool hist_ready,
                         bool guessed = false) {
  Scratch& s = c->s;
  const int rc = enqueue_topk_rows(c, tab, w, n, k, idx_rows, val_rows, hist_ready, guessed);
  if (rc) return rc;
  PtrTable vtab;
  for (int i = 0; i < kMaxW; ++i) vtab.p[i] = (i < w) ? val_rows + (size_t)i * (size_t)k : nullptr;
  int nblk = (int)((k + 256 * 16 - 1) / (256 * 16));
  if (nblk < 1) nblk = 1;
  if (nblk > kMaxChunks) nblk = kMaxChunks;
  hipLaunchKernelGGL(k_squares<false>, dim3(nblk, w), dim3(256), 0, c->stream, vtab, (int64_t)0, 0, vtab, k, nblk, s.partials,
                     s.partials);
  hipLaunchKernelGGL(k_sqnorm, dim3(1), dim3(1024), 0, c->stream, s.partials, nblk, (int)w, s.var_scratch,
                     sqnorm_out, s.leader_dev, argmax_out);
  HIP_TRY(c, hipGetLastError());
  return ARTOPK_OK;
}

template <bool STATS, int T>
void launch_small_t(artopk_ctx* c, const SmallStep& a) {
  const dim3 grid((unsigned)(a.nchunks * a.groups)), block(T);
  if (c->g_type == ARTOPK_G_BF16)
    hipLaunchKernelGGL((k_small_step<STATS, kGBF16, T>), grid, block, 0, c->stream, a);
  else if (c->g_type == ARTOPK_G_F16)
    hipLaunchKernelGGL((k_small_step<STATS, kGF16, T>), grid, block, 0, c->stream, a);
  else
    hipLaunchKernelGGL((k_small_step<STATS, kGF32, T>), grid, block, 0, c->stream, a);
}

template <bool STATS>
void launch_small(artopk_ctx* c, const SmallStep& a, int threads) {
  if (threads == 512) return launch_small_t<STATS, 512>(c, a);
  return launch_small_t<STATS, 1024>(c, a);
}

// Groups of workers that share out the first part of a short step: as many blocks as there are compute units.  Measured,
// us, variance rule, 1 / 2 / 4 / 8 / 16 groups: 65537 elements x 4 workers 29/26/23, x 8 39/32/28/25, x 16 61/46/35/31/30,
// x 64 195/127/84/63/62; 262143 x 8 45/36/32/33, x 16 69/52/44/45/52, x 64 232/152/122/118/128; 500009 x 8 45/42/49/57, x
// 16 70/65/68/79; 786427 x 8 49/59, x 16 77/94.  With a leader known up front the others' sums are formed while the block
// waits, unless they are many: 65537 x 8 22/-/23/22, x 16 27/-/28/26/26, x 64 64/-/60/45/47; 100003 x 64 87/-/63/55/56;
// 262143 x 16 36/-/38/40/45; 150001 x 64 one group and as many as there are units for 86/68, x 48 67/62, x 40 54/52, x
// 24 37/37, 200003 x 33 57/61, x 48 83/81.
int32_t small_groups(int32_t w, int64_t n, int32_t nchunks, bool known) {
  if (known && (w <= 16 || n > (w <= 40 ? (int64_t)128 << 10 : (int64_t)160 << 10))) return 1;
  return std::max<int32_t>(1, std::min<int32_t>(w, kSmallMaxUnits / nchunks));
}

// A flat step on a short vector in one launch.  leader >= 0: known up front; else it comes from the statistics
// (stats 1 or 2) or is in leader_dev already (stats 0).
int small_step(artopk_ctx* ctx, const PtrTable& gt, const PtrTable& rt, int32_t w, int64_t n, int64_t k, int stats,
               int leader, int32_t* leader_out, double* var_out, int32_t* idx_out, float* vals_out, float* sum_out,
               float* update_out) {
  Scratch& s = ctx->s;
  const int threads = n <= ((int64_t)1 << 20) ? 512 : 1024;
  SmallStep a{};
  a.g = gt;
  a.res = rt;
  a.n = n;
  a.k = (uint32_t)k;
  a.w_count = w;
  a.leader = leader;
  a.nchunks = (int32_t)((n + 8 * threads - 1) / (8 * threads));
  a.reps = a.nchunks <= 128 ? 1 : 2;
  a.groups = small_groups(w, n, a.nchunks, leader >= 0);
  a.raw_stats = stats == 2;
  a.list_cap = s.cap < (uint64_t)n ? s.cap : (uint32_t)n;
  a.ss = s.small;
  a.partials = s.partials;
  a.st = reinterpret_cast<SelState*>(s.zero_base + kSegState);
  a.err = s.err_dev;
  a.leader_dev = s.leader_dev;
  a.leader_out = (leader >= 0 || stats != 0) ? leader_out : nullptr;
  a.var_out = var_out;
  a.idx_out = idx_out;
  a.vals = vals_out;
  a.sum_out = sum_out;
  a.update = update_out;
  prof_dom(ctx, false);
  if (stats == 0)
    launch_small<false>(ctx, a, threads);
  else
    launch_small<true>(ctx, a, threads);
  HIP_TRY(ctx, hipGetLastError());
  prof_dom(ctx, true);
  for (int mark = 1; mark <= 4; ++mark) prof_mark(ctx, mark);
  return ARTOPK_OK;
}

}  // namespace

namespace {

// Zeroes the part of the short steps' scratch that is zero between steps.
void clear_small(artopk_ctx* c) {
  hipLaunchKernelGGL(k_fill_zero, dim3(64), dim3(256), 0, c->stream, c->s.small.hist, c->s.small_words, (uint32_t*)nullptr,
                     (size_t)0, (uint32_t*)nullptr, (size_t)0, 0, (int32_t*)nullptr, (int32_t*)nullptr);
}

// Where everything lies in the one allocation of a context.
struct Layout {
  uint32_t cap = 0;
  int64_t list_entries = 0, max_tiles = 0, mask_stride = 0, tilebuf_entries = 0;
  int64_t map_tiles = 0;
  int32_t blocks = 0;  // scratch blocks: one per segment, or per vector of a batch
  size_t o_hall = 0, o_mask = 0, o_zero = 0, o_S = 0, o_coff = 0, o_part = 0, o_var = 0, o_leader = 0, o_err = 0, o_counter = 0, o_list = 0, o_vals = 0, o_rows = 0, o_table = 0, o_cmap = 0, o_tstart = 0, o_tmap = 0, o_tbuf = 0, o_small = 0;
  size_t small_words = 0;  // words of the short vectors' scratch that have to be zero between steps
  size_t total = 0;
};

bool valid_limits(int32_t max_w, int64_t max_n, int64_t max_k, int32_t max_segments) {
  return !(max_w < 1 || max_w > ARTOPK_MAX_WORKERS || max_n < 1 || max_n >= (1ll << 31) || max_k < 1 ||
           max_k > max_n || max_segments < 1 || max_segments > 65535);
}

Layout scratch_layout(int32_t max_w, int64_t max_n, int64_t max_k, int32_t max_segments) {
  Layout L;
  // list capacity: every key above the range (< k of them) plus a generous share of candidates
  // (vectors of up to 4 Mi elements fit the list whole: their selection never needs the deeper
  // array passes, which are then not even launched)
  int64_t cand_share = max_n / 8;
  if (cand_share < ((int64_t)1 << 22)) cand_share = (int64_t)1 << 22;
  int64_t cap = max_k + cand_share;
  if (cap > max_n) cap = max_n;
  L.cap = (uint32_t)cap;
  // segmented layouts add per-segment rounding: n_s/8 may be raised to 4096 and bases are aligned
  L.list_entries = (int64_t)align_up((size_t)cap + (size_t)max_segments * 4100, kCompactTile) + kCompactTile;
  // a range [lo, hi) touches at most ceil(len / tile) + 1 look-back tiles
  // (or a batch of whole vectors)
  const int64_t batch = max_w < kMaxBatch ? max_w : kMaxBatch;
  const int64_t vec_tiles = (max_n + kCompactTile - 1) / kCompactTile;
  L.max_tiles = vec_tiles + 2 * (int64_t)max_segments + 1;
  if (L.max_tiles < vec_tiles * batch) L.max_tiles = vec_tiles * batch;
  L.blocks = max_segments > batch ? max_segments : (int32_t)batch;

  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off = align_up(off + bytes, 256);
    return o;
  };
  // zeroed region: one block per segment, then the look-back flags
  L.o_hall = take((size_t)max_w * kSlotWords * sizeof(uint32_t));
  // one bit per element and worker, in rows of 256 elements (whole tiles of the fused pass)
  L.mask_stride = (max_n + kPassTile - 1) / kPassTile * (kPassTile / 64);
  L.o_mask = take((size_t)max_w * (size_t)L.mask_stride * sizeof(uint64_t));
  L.o_zero = take((size_t)L.blocks * kSegWords * sizeof(uint32_t) +
                             (size_t)L.max_tiles * kNumLookback * sizeof(uint64_t));
  L.o_S = take(((size_t)max_w * kMaxChunks + (size_t)max_segments) * kHistBins * sizeof(uint32_t));
  L.o_coff = take(((size_t)kMaxChunks * (size_t)batch + (size_t)max_segments) * sizeof(uint32_t));
  L.o_part = take((size_t)max_w * kMaxPassBlocks * 3 * sizeof(double));
  L.o_var = take((size_t)max_w * sizeof(double));
  L.o_leader = take(sizeof(int32_t));
  L.o_err = take(sizeof(uint32_t));
  L.o_counter = take(sizeof(uint64_t));
  L.o_list = take((size_t)L.list_entries * sizeof(uint2));
  L.o_vals = take((size_t)max_w * (size_t)max_k * sizeof(float));
  L.o_rows = take((size_t)max_w * (size_t)max_k * sizeof(int32_t));
  L.o_table = take((size_t)max_segments * sizeof(SegDesc));
  L.o_cmap = take(((size_t)kMaxChunks + (size_t)max_segments) * sizeof(uint32_t));
  L.o_tstart = take((size_t)(max_n / kPassTile + 2) * sizeof(int32_t));
  // tiles of a segmented layout: two more than its share of the vector for every segment, and their groups
  const int64_t mark_tiles = max_n / kMarkTile + 1;
  L.map_tiles = max_segments > 1 ? mark_tiles + 2 * std::min<int64_t>(max_segments, mark_tiles) : 0;
  L.o_tmap = take((size_t)(L.map_tiles + L.map_tiles / 2 + 1) * sizeof(uint4));
  // pieces of marked elements: 6144 entries for every tile of the streaming passes (1.5 bytes per element)
  L.tilebuf_entries = (max_n + kPassTile - 1) / kPassTile * 6144;
  static_assert(piece_at(kPassTile) == 6144, "pieces lie as their elements do");
  L.o_tbuf = take((size_t)L.tilebuf_entries * sizeof(uint2));
  // (hist, ctr, claim, dig1 and dig2 have to be zero between steps)
  L.small_words = (size_t)(max_w + 1) * kSmallReps * kHistBins + kSmallCtr + kSmallMaxUnits + 2 * kSmallReps * 128;
  const int64_t small_n = max_n < kSmallMaxNLimit ? max_n : kSmallMaxNLimit;
  size_t small_bytes = (L.small_words + (size_t)kSmallMaxChunks * 129) * sizeof(uint32_t);
  // (callers plan with the size that the header states)
  const size_t stated = (size_t)max_w * ((size_t)128 << 10) + (size_t)(4.5 * (double)small_n) + ((size_t)1184 << 10);
  if (small_bytes < stated) small_bytes = stated;
  L.o_small = take(small_bytes);
  L.total = off;
  return L;
}

}  // namespace

extern "C" {

int32_t artopk_version(void) { return 200; }  // 0.2.0: options, counted round-robin leader, allocation-free variance

const char* artopk_last_error(const artopk_ctx* ctx) { return ctx ? ctx->err : g_noctx_err; }

int artopk_create(artopk_ctx** out, int32_t max_w, int64_t max_n, int64_t max_k, int32_t max_segments,
                  void* hip_stream) {
  if (!out) return ARTOPK_EINVAL;
  if (!valid_limits(max_w, max_n, max_k, max_segments)) return ARTOPK_EINVAL;
  artopk_ctx* c = new (std::nothrow) artopk_ctx();
  if (!c) return ARTOPK_ENOMEM;
  c->stream = reinterpret_cast<hipStream_t>(hip_stream);
  c->max_w = max_w;
  c->max_n = max_n;
  c->max_k = max_k;
  c->max_seg = max_segments;
  hipError_t e = hipGetDevice(&c->device);
  int cus = 0;
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, c->device);
  if (e != hipSuccess) {
    delete c;
    return ARTOPK_EHIP;
  }
  c->num_cu = cus > 0 ? cus : 256;

  Scratch& s = c->s;
  const Layout L = scratch_layout(max_w, max_n, max_k, max_segments);
  s.cap = L.cap;
  s.list_entries = L.list_entries;
  s.max_tiles = L.max_tiles;
  s.mask_stride = L.mask_stride;
  s.tilebuf_entries = L.tilebuf_entries;
  const size_t total = L.total;

  e = hipMalloc(&c->slab, total);
  if (e != hipSuccess) {
    delete c;
    return ARTOPK_ENOMEM;
  }
  char* base = static_cast<char*>(c->slab);
  s.h_all = reinterpret_cast<uint32_t*>(base + L.o_hall);
  s.mask = reinterpret_cast<uint64_t*>(base + L.o_mask);
  s.zero_base = reinterpret_cast<uint32_t*>(base + L.o_zero);
  // kSegWords is even, so the flags stay 8-byte aligned
  s.flags = reinterpret_cast<uint64_t*>(s.zero_base + (size_t)L.blocks * kSegWords);
  s.S = reinterpret_cast<uint32_t*>(base + L.o_S);
  s.chunk_off = reinterpret_cast<uint32_t*>(base + L.o_coff);
  s.partials = reinterpret_cast<double*>(base + L.o_part);
  s.var_scratch = reinterpret_cast<double*>(base + L.o_var);
  s.leader_dev = reinterpret_cast<int32_t*>(base + L.o_leader);
  s.err_dev = reinterpret_cast<uint32_t*>(base + L.o_err);
  s.counter_dev = reinterpret_cast<uint64_t*>(base + L.o_counter);
  s.list = reinterpret_cast<uint2*>(base + L.o_list);
  s.vals = reinterpret_cast<float*>(base + L.o_vals);
  s.idx_rows = reinterpret_cast<int32_t*>(base + L.o_rows);
  s.table_dev = reinterpret_cast<SegDesc*>(base + L.o_table);
  s.chunk_map = reinterpret_cast<uint32_t*>(base + L.o_cmap);
  s.tile_start = reinterpret_cast<int32_t*>(base + L.o_tstart);
  s.tile_map = reinterpret_cast<uint4*>(base + L.o_tmap);
  s.map_tiles = L.map_tiles;
  s.tilebuf = reinterpret_cast<uint2*>(base + L.o_tbuf);

  uint32_t* small = reinterpret_cast<uint32_t*>(base + L.o_small);
  s.small.hist = small;
  s.small.ctr = small + (size_t)max_w * kSmallReps * kHistBins;
  s.small.claim = s.small.ctr + kSmallCtr;
  s.small.dig1 = s.small.claim + kSmallMaxUnits;
  s.small.dig2 = s.small.dig1 + (size_t)kSmallReps * kHistBins;
  s.small.above = s.small.dig2 + 2 * kSmallReps * 128;
  s.small.rows = s.small.above + kSmallMaxChunks;
  s.small_words = L.small_words;

  // leader, error word and step counter start at zero (stream-ordered before any later call)
  hipLaunchKernelGGL(k_fill_zero, dim3(1), dim3(256), 0, c->stream,
                     reinterpret_cast<uint32_t*>(s.leader_dev), (size_t)1, s.err_dev, (size_t)1,
                     reinterpret_cast<uint32_t*>(s.counter_dev), (size_t)2, 0, (int32_t*)nullptr,
                     (int32_t*)nullptr);
  clear_small(c);
  if (hipGetLastError() != hipSuccess) {
    (void)hipFree(c->slab);
    delete c;
    return ARTOPK_EHIP;
  }
  *out = c;
  return ARTOPK_OK;
}

int64_t artopk_scratch_bytes(int32_t max_w, int64_t max_n, int64_t max_k, int32_t max_segments) {
  if (!valid_limits(max_w, max_n, max_k, max_segments)) return -1;
  return (int64_t)scratch_layout(max_w, max_n, max_k, max_segments).total;
}

int artopk_destroy(artopk_ctx* ctx) {
  if (!ctx) return ARTOPK_EINVAL;
  if (ctx->ev_created)
    for (int r = 0; r < artopk_ctx::kRing; ++r)
      for (int i = 0; i < artopk_ctx::kMarks; ++i)
        if (ctx->ev[r][i]) (void)hipEventDestroy(ctx->ev[r][i]);
  if (ctx->slab) (void)hipFree(ctx->slab);
  delete ctx;
  return ARTOPK_OK;
}

int artopk_status(artopk_ctx* ctx) {
  if (!ctx) return ARTOPK_EINVAL;
  HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
  uint32_t err = 0;
  HIP_TRY(ctx, hipMemcpy(&err, ctx->s.err_dev, sizeof(err), hipMemcpyDeviceToHost));
  if (err) {
    uint32_t zero = 0;
    clear_small(ctx);  // (a short step may have ended before its scratch was zero again)
    HIP_TRY(ctx, hipGetLastError());
    HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
    HIP_TRY(ctx, hipMemcpy(ctx->s.err_dev, &zero, sizeof(zero), hipMemcpyHostToDevice));
    return fail(ctx, ARTOPK_ESTATE, "device error word 0x%x (1 = histogram/count mismatch, 2 = scan wait expired, 4 = kernel sequence, 8 = index out of range)", err);
  }
  return ARTOPK_OK;
}

int artopk_set_profile(artopk_ctx* ctx, int32_t enable) {
  if (!ctx) return ARTOPK_EINVAL;
  if (enable && !ctx->ev_created) {
    for (int r = 0; r < artopk_ctx::kRing; ++r)
      for (int i = 0; i < artopk_ctx::kMarks; ++i) HIP_TRY(ctx, hipEventCreate(&ctx->ev[r][i]));
    ctx->ev_created = true;
  }
  ctx->profile = enable != 0;
  ctx->profile_level = enable;
  ctx->prof_calls = 0;
  for (int r = 0; r < artopk_ctx::kRing; ++r)
    for (int i = 0; i < artopk_ctx::kMarks; ++i) ctx->ev_valid[r][i] = false;
  return ARTOPK_OK;
}

int artopk_set_option(artopk_ctx* ctx, int32_t key, int64_t value) {
  if (!ctx) return ARTOPK_EINVAL;
  switch (key) {
    case ARTOPK_OPT_GUESS_MIN_N:
      if (value < 1 || value > (1ll << 31)) return fail(ctx, ARTOPK_EINVAL, "ARTOPK_OPT_GUESS_MIN_N outside [1, 2^31]");
      ctx->guess_min_n = value;
      ctx->guess_min_n_set = true;
      return ARTOPK_OK;
    case ARTOPK_OPT_UPDATE_TILES_MIN_N:
      if (value < 1 || value > (1ll << 31))
        return fail(ctx, ARTOPK_EINVAL, "ARTOPK_OPT_UPDATE_TILES_MIN_N outside [1, 2^31]");
      ctx->update_tiles_min_n = value;
      return ARTOPK_OK;
    case ARTOPK_OPT_LEADER_FIRST:
      if (value != 0 && value != 1) return fail(ctx, ARTOPK_EINVAL, "ARTOPK_OPT_LEADER_FIRST takes 0 or 1");
      ctx->leader_first = value != 0;
      return ARTOPK_OK;
    case ARTOPK_OPT_NONTEMPORAL:
      if (value != 0 && value != 1) return fail(ctx, ARTOPK_EINVAL, "ARTOPK_OPT_NONTEMPORAL takes 0 or 1");
      ctx->pass_a_nt = value != 0;
      return ARTOPK_OK;
    case ARTOPK_OPT_STAGE_TILES:
      if (value < 0 || value > 2) return fail(ctx, ARTOPK_EINVAL, "ARTOPK_OPT_STAGE_TILES takes 0, 1 or 2");
      ctx->stage_tiles = (int)value;
      return ARTOPK_OK;
    case ARTOPK_OPT_SHORT_MAX_N:
      if (value < 0 || value > kSmallMaxNLimit) return fail(ctx, ARTOPK_EINVAL, "ARTOPK_OPT_SHORT_MAX_N outside [0, 2^21]");
      ctx->small_max_n = value;
      ctx->small_max_n_set = true;
      return ARTOPK_OK;
    default:
      return fail(ctx, ARTOPK_EINVAL, "unknown option %d", key);
  }
}

int artopk_get_option(const artopk_ctx* ctx, int32_t key, int64_t* value_out) {
  if (!ctx || !value_out) return ARTOPK_EINVAL;
  switch (key) {
    case ARTOPK_OPT_GUESS_MIN_N: *value_out = ctx->guess_min_n; return ARTOPK_OK;
    case ARTOPK_OPT_UPDATE_TILES_MIN_N: *value_out = ctx->update_tiles_min_n; return ARTOPK_OK;
    case ARTOPK_OPT_LEADER_FIRST: *value_out = ctx->leader_first ? 1 : 0; return ARTOPK_OK;
    case ARTOPK_OPT_NONTEMPORAL: *value_out = ctx->pass_a_nt ? 1 : 0; return ARTOPK_OK;
    case ARTOPK_OPT_STAGE_TILES: *value_out = ctx->stage_tiles; return ARTOPK_OK;
    case ARTOPK_OPT_SHORT_MAX_N: *value_out = ctx->small_max_n; return ARTOPK_OK;
    default: return ARTOPK_EINVAL;
  }
}

// Reads back the selection state of segment 0 as the last step left it.
int artopk_select_info(artopk_ctx* ctx, int32_t* info_out, int32_t count) {
  if (!ctx || !info_out || count < 0) return ARTOPK_EINVAL;
  HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
  SelState st{};
  HIP_TRY(ctx, hipMemcpy(&st, ctx->s.zero_base + kSegState, sizeof(st), hipMemcpyDeviceToHost));
  int32_t bounds = 0;
  for (int32_t seg = 0; count > 9 && seg < ctx->last_tiles; seg += 64) {
    SelState of[64];
    const int32_t some = std::min(ctx->last_tiles - seg, 64);
    HIP_TRY(ctx, hipMemcpy2D(of, sizeof(SelState), ctx->s.zero_base + (size_t)seg * kSegWords + kSegState,
                             kSegWords * sizeof(uint32_t), sizeof(SelState), (size_t)some, hipMemcpyDeviceToHost));
    for (int32_t i = 0; i < some; ++i) bounds += of[i].use_mask != 0u ? 1 : 0;
  }
  const int32_t v[10] = {ctx->last_guessed, ctx->last_guessed ? (int32_t)st.use_mask : 0, (int32_t)st.list_count,
                         (int32_t)st.compact_level, ctx->last_dom_workers, ctx->last_short,
                         ctx->last_short ? (int32_t)st.many : 0, ctx->last_one_launch, ctx->last_tiles > 0 ? 1 : 0, bounds};
  for (int i = 0; i < count && i < 10; ++i) info_out[i] = v[i];
  return ARTOPK_OK;
}

// Averages every stage over the calls recorded since profiling was enabled
// (at most the kRing most recent ones).
int artopk_get_profile(artopk_ctx* ctx, float* ms_out, int32_t count) {
  if (!ctx || !ms_out || count < 0) return ARTOPK_EINVAL;
  if (!ctx->ev_created) return fail(ctx, ARTOPK_EINVAL, "profiling was never enabled");
  HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
  double acc[ARTOPK_PROF_COUNT] = {0, 0, 0, 0, 0};
  int cnt[ARTOPK_PROF_COUNT] = {0, 0, 0, 0, 0};
  for (int r = 0; r < artopk_ctx::kRing; ++r) {
    const bool* v = ctx->ev_valid[r];
    for (int i = 0; i < 4; ++i) {
      if (v[i] && v[i + 1]) {
        float ms = 0.f;
        HIP_TRY(ctx, hipEventElapsedTime(&ms, ctx->ev[r][i], ctx->ev[r][i + 1]));
        acc[i] += ms;
        cnt[i]++;
      }
    }
    int last = -1;
    for (int i = 4; i >= 1; --i)
      if (v[i]) {
        last = i;
        break;
      }
    if (v[0] && last > 0) {
      float ms = 0.f;
      HIP_TRY(ctx, hipEventElapsedTime(&ms, ctx->ev[r][0], ctx->ev[r][last]));
      acc[ARTOPK_PROF_TOTAL] += ms;
      cnt[ARTOPK_PROF_TOTAL]++;
    }
  }
  for (int i = 0; i < count && i < ARTOPK_PROF_COUNT; ++i) ms_out[i] = cnt[i] ? (float)(acc[i] / cnt[i]) : 0.f;
  return ARTOPK_OK;
}

int artopk_variance(artopk_ctx* ctx, const float* const* x, int32_t w, int64_t n, double* var_out,
                    int32_t* argmax_out) {
  int rc = check_common(ctx, w, n, 1);
  if (rc) return rc;
  if ((rc = check_ptr_table(ctx, x, w, "x"))) return rc;
  if (!var_out) return fail(ctx, ARTOPK_EINVAL, "var_out is NULL");
  {
    RangeSet rs;
    rs.add_table(reinterpret_cast<const void* const*>(x), w, (size_t)n * 4, false, "x");
    rs.add(var_out, (size_t)w * 8, true, "var_out");
    rs.add(argmax_out, 4, true, "argmax_out");
    if ((rc = rs.check(ctx))) return rc;
  }
  const PtrTable tab = make_table(x, w);
  const int nblk = stats_blocks(ctx->num_cu, w, n);
  Scratch& s = ctx->s;
  launch_stats(ctx->stream, tab, nblk, w, n, s.partials);
  hipLaunchKernelGGL(k_leader, dim3(1), dim3(1024), 0, ctx->stream, s.partials, (int)w, nblk, n, s.var_scratch,
                     var_out, s.leader_dev, argmax_out);
  HIP_TRY(ctx, hipGetLastError());
  return ARTOPK_OK;
}

namespace {

// Per-device address of the fixed scratch and the device's compute-unit count, looked up the
// first time artopk_variance_static runs with that device current.
struct StaticDevice {
  bool ready = false;
  double* ptr = nullptr;
  int num_cu = 0;
};
constexpr int kMaxDevices = 64;
StaticDevice g_static_dev[kMaxDevices];
std::mutex g_static_mu;

int static_device(const StaticDevice** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(nullptr, ARTOPK_EHIP, "hipGetDevice failed: %s", hipGetErrorString(e));
  if (dev < 0 || dev >= kMaxDevices) return fail(nullptr, ARTOPK_EINVAL, "device %d outside [0, %d)", dev, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_static_mu);
  StaticDevice& sd = g_static_dev[dev];
  if (!sd.ready) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || p == nullptr)
      return fail(nullptr, ARTOPK_EHIP, "hipGetSymbolAddress(scratch) failed on device %d: %s", dev,
                  hipGetErrorString(e));
    int cus = 0;
    e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return fail(nullptr, ARTOPK_EHIP, "hipDeviceGetAttribute failed: %s", hipGetErrorString(e));
    sd.ptr = static_cast<double*>(p);
    sd.num_cu = cus > 0 ? cus : 256;
    sd.ready = true;
  }
  *out = &sd;
  return ARTOPK_OK;
}

}  // namespace

int artopk_variance_static(const float* const* x, int32_t w, int64_t n, double* var_out, int32_t* argmax_out,
                           void* hip_stream) {
  if (w < 1 || w > ARTOPK_MAX_WORKERS)
    return fail(nullptr, ARTOPK_EINVAL, "W=%d outside [1, %d] (the fixed scratch holds %d workers)", w,
                ARTOPK_MAX_WORKERS, ARTOPK_MAX_WORKERS);
  if (n < 1 || n >= (1ll << 31)) return fail(nullptr, ARTOPK_EINVAL, "N=%lld outside [1, 2^31)", (long long)n);
  int rc = check_ptr_table(nullptr, x, w, "x");
  if (rc) return rc;
  if (!var_out) return fail(nullptr, ARTOPK_EINVAL, "var_out is NULL");
  {
    RangeSet rs;
    rs.add_table(reinterpret_cast<const void* const*>(x), w, (size_t)n * 4, false, "x");
    rs.add(var_out, (size_t)w * 8, true, "var_out");
    rs.add(argmax_out, 4, true, "argmax_out");
    if ((rc = rs.check(nullptr))) return rc;
  }
  const StaticDevice* sd = nullptr;
  if ((rc = static_device(&sd))) return rc;
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  const PtrTable tab = make_table(x, w);
  const int nblk = stats_blocks(sd->num_cu, w, n);  // <= kMaxChunks, so w * nblk * 3 <= kStaticPartials
  double* partials = sd->ptr;
  double* var_scratch = sd->ptr + kStaticPartials;
  int32_t* leader_word = reinterpret_cast<int32_t*>(sd->ptr + kStaticPartials + kMaxW);
  // every word of the scratch that is read is written first by these two launches: nothing to clear
  launch_stats(st, tab, nblk, w, n, partials);
  hipLaunchKernelGGL(k_leader, dim3(1), dim3(1024), 0, st, partials, (int)w, nblk, n, var_scratch, var_out,
                     leader_word, argmax_out);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(nullptr, ARTOPK_EHIP, "kernel launch failed: %s", hipGetErrorString(e));
  return ARTOPK_OK;
}

int artopk_select_topk(artopk_ctx* ctx, const float* acc, int64_t n, int32_t nseg, const int64_t* seg_off,
                       const int64_t* seg_k, int64_t k, int32_t* idx_out) {
  int rc = check_common(ctx, 1, n, k);
  if (rc) return rc;
  if (!acc || !aligned16(acc)) return fail(ctx, ARTOPK_EINVAL, "acc is NULL or not 16-byte aligned");
  if (!idx_out) return fail(ctx, ARTOPK_EINVAL, "idx_out is NULL");
  if ((rc = check_segments(ctx, n, nseg, seg_off, seg_k, k))) return rc;
  {
    RangeSet rs;
    rs.add(acc, (size_t)n * 4, false, "acc");
    rs.add(idx_out, (size_t)k * 4, true, "idx_out");
    if ((rc = rs.check(ctx))) return rc;
  }
  const float* one[1] = {acc};
  const PtrTable tab = make_table(one, 1);
  prof_begin(ctx);
  prof_mark(ctx, 1);
  ctx->last_guessed = 0;
  ctx->last_dom_workers = 1;
  ctx->last_short = 0;
  if (seg_off && nseg > 1) {
    const Plan* pl = nullptr;
    if ((rc = segmented_plan(ctx, n, nseg, seg_off, seg_k, &pl))) return rc;
    if ((rc = enqueue_clear(ctx, *pl, 0, 0, nullptr, segments_by_tiles(ctx, *pl, n)))) return rc;  // the single vector is "leader 0"
    rc = segments_by_tiles(ctx, *pl, n) ? enqueue_tiles(ctx, *pl, tab, n, idx_out, nullptr, GuessPlan{}, nullptr, nullptr, false)
                                             : enqueue_select(ctx, *pl, tab, n, idx_out, false, 0);
  } else {
    rc = enqueue_topk_rows(ctx, tab, 1, n, k, idx_out, nullptr, false, false);
  }
  prof_mark(ctx, 2);
  return rc;
}

int artopk_gather_sum(artopk_ctx* ctx, const float* const* acc, int32_t w, int64_t n, const int32_t* idx,
                      int64_t k, float* vals_out, float* sum_out) {
  int rc = check_common(ctx, w, n, k);
  if (rc) return rc;
  if ((rc = check_ptr_table(ctx, acc, w, "acc"))) return rc;
  if (!idx || !sum_out) return fail(ctx, ARTOPK_EINVAL, "idx or sum_out is NULL");
  {
    RangeSet rs;
    rs.add_table(reinterpret_cast<const void* const*>(acc), w, (size_t)n * 4, false, "acc");
    rs.add(idx, (size_t)k * 4, false, "idx");
    rs.add(vals_out, (size_t)w * (size_t)k * 4, true, "vals_out");
    rs.add(sum_out, (size_t)k * 4, true, "sum_out");
    if ((rc = rs.check(ctx))) return rc;
  }
  const PtrTable tab = make_table(acc, w);
  return enqueue_gather(ctx, tab, w, n, idx, k, vals_out, sum_out, false);
}

int artopk_scatter_residual(artopk_ctx* ctx, float* const* residual, int32_t w, int64_t n, const int32_t* idx,
                            int64_t k, const float* sum, float* update) {
  int rc = check_common(ctx, w, n, k);
  if (rc) return rc;
  if ((rc = check_ptr_table(ctx, residual, w, "residual"))) return rc;
  if (!idx || !sum || !update) return fail(ctx, ARTOPK_EINVAL, "idx, sum or update is NULL");
  if (!aligned16(update)) return fail(ctx, ARTOPK_EINVAL, "update is not 16-byte aligned");
  {
    RangeSet rs;
    rs.add_table(reinterpret_cast<const void* const*>(residual), w, (size_t)n * 4, true, "residual");
    rs.add(idx, (size_t)k * 4, false, "idx");
    rs.add(sum, (size_t)k * 4, false, "sum");
    rs.add(update, (size_t)n * 4, true, "update");
    if ((rc = rs.check(ctx))) return rc;
  }
  const PtrTable tab = make_table(residual, w);
  const int blocks = (int)((k + 255) / 256);
  hipLaunchKernelGGL(k_zero_at, dim3(blocks), dim3(256), 0, ctx->stream, tab, (int)w, n, idx, k, ctx->s.err_dev);
  HIP_TRY(ctx, hipGetLastError());
  return enqueue_update_fill(ctx, update, n, idx, sum, k);
}

int artopk_topk_workers(artopk_ctx* ctx, const float* const* acc, int32_t w, int64_t n, int64_t k,
                        int32_t* idx_out, float* vals_out, double* sqnorm_out, int32_t* argmax_out) {
  int rc = check_common(ctx, w, n, k);
  if (rc) return rc;
  if ((rc = check_ptr_table(ctx, acc, w, "acc"))) return rc;
  if (!idx_out) return fail(ctx, ARTOPK_EINVAL, "idx_out is NULL");
  {
    RangeSet rs;
    rs.add_table(reinterpret_cast<const void* const*>(acc), w, (size_t)n * 4, false, "acc");
    rs.add(idx_out, (size_t)w * (size_t)k * 4, true, "idx_out");
    rs.add(vals_out, (size_t)w * (size_t)k * 4, true, "vals_out");
    rs.add(sqnorm_out, (size_t)w * 8, true, "sqnorm_out");
    rs.add(argmax_out, 4, true, "argmax_out");
    if ((rc = rs.check(ctx))) return rc;
  }
  const PtrTable tab = make_table(acc, w);
  return enqueue_topk_workers(ctx, tab, w, n, k, idx_out, vals_out ? vals_out : ctx->s.vals, sqnorm_out,
                              argmax_out, false);
}

int artopk_compression_gain(artopk_ctx* ctx, const float* const* residual, int32_t w, int64_t n,
                            const float* vals, int64_t k, double* gain_out) {
  int rc = check_common(ctx, w, n, k);
  if (rc) return rc;
  if ((rc = check_ptr_table(ctx, residual, w, "residual"))) return rc;
  if (!vals || !gain_out) return fail(ctx, ARTOPK_EINVAL, "vals or gain_out is NULL");
  {
    RangeSet rs;
    rs.add_table(reinterpret_cast<const void* const*>(residual), w, (size_t)n * 4, false, "residual");
    rs.add(vals, (size_t)w * (size_t)k * 4, false, "vals");
    rs.add(gain_out, (size_t)w * 8, true, "gain_out");
    if ((rc = rs.check(ctx))) return rc;
  }
  Scratch& s = ctx->s;
  const PtrTable rtab = make_table(residual, w);
  PtrTable vtab;
  for (int i = 0; i < kMaxW; ++i) vtab.p[i] = (i < w) ? const_cast<float*>(vals) + (size_t)i * (size_t)k : nullptr;
  const int nblk_res = stats_blocks(ctx->num_cu, w, n);
  int nblk_vals = (int)((k + 256 * 16 - 1) / (256 * 16));
  if (nblk_vals < 1) nblk_vals = 1;
  if (nblk_vals > kMaxChunks / 2) nblk_vals = kMaxChunks / 2;
  // the two partial arrays share the variance scratch: residual partials first
  double* part_res = s.partials;
  double* part_vals = s.partials + (size_t)ctx->max_w * (kMaxChunks / 2);
  const int nblk_res_c = nblk_res > kMaxChunks / 2 ? kMaxChunks / 2 : nblk_res;
  const dim3 grid((unsigned)(nblk_vals + nblk_res_c), (unsigned)w);
  if (beyond_cache(w, n))
    hipLaunchKernelGGL(k_squares<true>, grid, dim3(256), 0, ctx->stream, rtab, n, nblk_res_c, vtab, k, nblk_vals, part_res,
                       part_vals);
  else
    hipLaunchKernelGGL(k_squares<false>, grid, dim3(256), 0, ctx->stream, rtab, n, nblk_res_c, vtab, k, nblk_vals, part_res,
                       part_vals);
  hipLaunchKernelGGL(k_gain, dim3(1), dim3(1024), 0, ctx->stream, part_vals, nblk_vals, part_res, nblk_res_c, (int)w,
                     gain_out);
  HIP_TRY(ctx, hipGetLastError());
  return ARTOPK_OK;
}

int artopk_apply_update(artopk_ctx* ctx, float* weights, int64_t n, const int32_t* idx, const float* sum,
                        int64_t k, float eta) {
  int rc = check_common(ctx, 1, n, k);
  if (rc) return rc;
  if (!weights || !idx || !sum) return fail(ctx, ARTOPK_EINVAL, "weights, idx or sum is NULL");
  {
    RangeSet rs;
    rs.add(weights, (size_t)n * 4, true, "weights");
    rs.add(idx, (size_t)k * 4, false, "idx");
    rs.add(sum, (size_t)k * 4, false, "sum");
    if ((rc = rs.check(ctx))) return rc;
  }
  const int blocks = (int)((k + 255) / 256);
  hipLaunchKernelGGL(k_apply_update, dim3(blocks), dim3(256), 0, ctx->stream, weights, n, idx, sum, k, eta,
                     ctx->s.err_dev);
  HIP_TRY(ctx, hipGetLastError());
  return ARTOPK_OK;
}

namespace {

// Blocks per worker of a pass A that strides over the tiles of n elements, or 0 where it had better take chunks: a quarter
// of a tile each, they still fill the chip (variance rule, us a step, one in a hundred and in ten kept, chunks / tiles,
// normal values and sorted ones, whose digits all are a tile's: 37 tiles of all workers, 1.2 M x 1, 51/52 57/64, 68/88
// 68/88; 68, 1.1 M x 2, 59/55 66/65, 81/89 80/89; 128, 1 M x 4, 64/57 71/67, 83/90 83/90; 160, 1.3 M x 4, 72/59 81/71, 96/91
// 95/90; 232, 1.9 M x 4, 84/65 95/79, 111/94 109/93).  512 / 1024 / 2048 blocks over all workers: 11.7 M x 8
// 292.7/288.4/286.8 us a step, 5 M x 16 258/260/249.
int tile_blocks(int64_t n, int workers) {
  const int64_t ntiles = (n + kPassTile - 1) / kPassTile;
  if (ntiles * workers < 128) return 0;
  const int64_t blocks = 2048 / workers;
  return (int)(ntiles < blocks ? ntiles : blocks);
}

// One step; the g rows hold elements of type g_type (float32 rows are passed as they are, 16-bit
// rows behind the same pointer type).
int step_impl(artopk_ctx* ctx, const float* const* g, int32_t g_type, float* const* residual, int32_t w, int64_t n,
              int32_t nseg, const int64_t* seg_off, const int64_t* seg_k, int64_t k, int32_t mode,
              uint64_t step, int32_t fixed_leader, int32_t* leader_out, double* var_out, int32_t* idx_out,
              float* vals_out, float* sum_out, float* update_out) {
  int rc = check_common(ctx, w, n, k);
  if (rc) return rc;
  if (g_type != ARTOPK_G_F32 && g_type != ARTOPK_G_BF16 && g_type != ARTOPK_G_F16)
    return fail(ctx, ARTOPK_EINVAL, "unknown gradient element type %d", g_type);
  ctx->g_type = g_type;
  if ((rc = check_ptr_table(ctx, g, w, "g", g_type == ARTOPK_G_F32 ? 16 : 8))) return rc;
  if ((rc = check_ptr_table(ctx, residual, w, "residual"))) return rc;
  if (!idx_out || !sum_out) return fail(ctx, ARTOPK_EINVAL, "idx_out or sum_out is NULL");
  if (update_out && !aligned16(update_out)) return fail(ctx, ARTOPK_EINVAL, "update_out is not 16-byte aligned");
  if ((rc = check_segments(ctx, n, nseg, seg_off, seg_k, k))) return rc;
  {
    RangeSet rs;
    rs.add_table(reinterpret_cast<const void* const*>(g), w, (size_t)n * (g_type == ARTOPK_G_F32 ? 4 : 2), false, "g");
    rs.add_table(reinterpret_cast<const void* const*>(residual), w, (size_t)n * 4, true, "residual");
    rs.add(leader_out, 4, true, "leader_out");
    rs.add(var_out, (size_t)w * 8, true, "var_out");
    rs.add(idx_out, (size_t)k * 4, true, "idx_out");
    rs.add(vals_out, (size_t)w * (size_t)k * 4, true, "vals_out");
    rs.add(sum_out, (size_t)k * 4, true, "sum_out");
    rs.add(update_out, (size_t)n * 4, true, "update_out");
    if ((rc = rs.check(ctx))) return rc;
  }
  int leader_host = -1;
  if (mode == ARTOPK_STAR) {
    leader_host = (int)(step % (uint64_t)w);
  } else if (mode == ARTOPK_FIXED) {
    if (fixed_leader < 0 || fixed_leader >= w) return fail(ctx, ARTOPK_EINVAL, "fixed_leader outside [0, W)");
    leader_host = fixed_leader;
  } else if (mode == ARTOPK_VAR_TOPK) {
    if (seg_off != nullptr && nseg > 1)
      return fail(ctx, ARTOPK_EINVAL, "ARTOPK_VAR_TOPK is defined for the unsegmented selection only");
  } else if (mode != ARTOPK_VAR && mode != ARTOPK_VAR_G && mode != ARTOPK_STAR_COUNTER) {
    return fail(ctx, ARTOPK_EINVAL, "unknown mode %d", mode);
  }
  // the leader is found on the device, from statistics of the pass or from the counter
  const bool device_leader = mode == ARTOPK_VAR || mode == ARTOPK_VAR_G || mode == ARTOPK_STAR_COUNTER;

  Scratch& s = ctx->s;
  hipStream_t st = ctx->stream;
  const PtrTable gt = make_table(g, w);
  const PtrTable rt = make_table(residual, w);
  const bool segmented = seg_off != nullptr && nseg > 1;
  // a flat selection on a long vector samples a threshold guess first; its chunks are then whole
  // tiles of the fused pass, which strides over the tiles and counts per chunk
  const bool leader_first = (mode == ARTOPK_STAR || mode == ARTOPK_FIXED) && ctx->leader_first;
  const GuessPlan gp = segmented ? GuessPlan{} : plan_guess(ctx, n, k, leader_first);
  Plan flat;
  const Plan* pl = &flat;
  if (segmented) {
    if ((rc = segmented_plan(ctx, n, nseg, seg_off, seg_k, &pl))) return rc;
  } else {
    flat = flat_plan(ctx, n, k, -1, gp.on);
  }
  // pass A always works on whole-vector chunks; for a flat select they are the select's chunks too, unless k_tail
  // selects, which needs none: then the pass strides over the tiles
  const ChunkGeom geom = make_geom(0, n, kMaxChunks, gp.on);
  // (sparse selections of few tiles: list kernels / k_tail, us, 1 M x 2, one in a thousand and in a hundred 50.8/51.8
  // 53.8/53.7, 1.3 M 57.6/61.0 61.5/61.5, 1.8 M 61.2/63.8 66.2/64.8; without statistics 1.3 M 53.5/56.5 59.1/57.2)
  flat.lists = device_leader && tile_blocks(n, (int)w) == 0 && 256 * k < n;
  const int tile_nblk = !segmented && !gp.on && !leader_first && mode != ARTOPK_VAR_TOPK && tail_plan(flat, n, kTailHist).ranges > 0
                            ? tile_blocks(n, (int)w) : 0;
  const bool by_tile = tile_nblk > 0;
  const int pass_nblk = by_tile ? tile_nblk : (int)geom.nchunks;
  const dim3 grid(pass_nblk, w);

  // a long segmented vector whose leader is found on the device: the fused pass strides over the tiles as on the guess
  // route (the selection reads the leader's vector again either way, by tiles or for its segments' histograms)
  const bool seg_stride = segmented && n >= ctx->guess_min_n;
  const bool by_tiles = segmented && segments_by_tiles(ctx, *pl, n);

  ctx->last_guessed = 0;
  ctx->last_dom_workers = w;
  ctx->last_short = 0;
  ctx->last_tiles = 0;
  if (mode == ARTOPK_VAR_TOPK) {
    // Literal Alg. 1: Top-k on every worker, leader = largest squared norm of its own k values,
    // then the leader's indices are the shared ones.
    prof_begin(ctx);
    prof_mark(ctx, 0);
    if ((rc = enqueue_clear(ctx, *pl, (int)w))) return rc;
    // every worker selects on its own vector: on long vectors every worker gets a guessed bound and
    // leaves a mask, as under the variance rule
    ctx->last_guessed = gp.on ? 1 : 0;
    ctx->lvl1_a = 0;
    ctx->lvl1_b = 1;
    if (gp.on) enqueue_guess(ctx, gp, gt, rt, (int)w);
    prof_dom(ctx, false);
    if (gp.on) {
      launch_pass_mark(ctx, 0, (int)w, gt, rt, n, geom.chunk_elems);
    } else {
      launch_pass_a(ctx, 0, 2, grid, gt, rt, n, geom, -1);
    }
    prof_dom(ctx, true);
    prof_mark(ctx, 1);
    if ((rc = enqueue_topk_workers(ctx, rt, w, n, k, s.idx_rows, s.vals, var_out, leader_out, true, gp.on))) return rc;
    hipLaunchKernelGGL(k_copy_i32, dim3((int)((k + 255) / 256)), dim3(256), 0, st, s.idx_rows, s.leader_dev, k,
                       idx_out);
    prof_mark(ctx, 2);
    if ((rc = enqueue_gather(ctx, rt, w, n, idx_out, k, vals_out, sum_out, true))) return rc;
    prof_mark(ctx, 3);
    if (update_out && (rc = enqueue_update_fill(ctx, update_out, n, idx_out, sum_out, k))) return rc;
    prof_mark(ctx, 4);
    return ARTOPK_OK;
  }

  const int64_t short_n = (device_leader && w < 8) ? ctx->small_max_n / 4 * 3 : ctx->small_max_n;
  const bool too_many = device_leader && mode != ARTOPK_STAR_COUNTER && !ctx->small_max_n_set && w > 24 &&
                        n >= kSmallManyMinN && n <= kSmallManyMaxN && (int64_t)w * n > kSmallMaxValues;
  if (!segmented && !gp.on && n <= short_n && !too_many && (leader_first || device_leader)) {
    ctx->lvl1_a = 0;
    ctx->lvl1_b = 1;
    prof_begin(ctx);
    prof_mark(ctx, 0);
    if (mode == ARTOPK_STAR_COUNTER) {
      hipLaunchKernelGGL(k_counter_leader, dim3(1), dim3(64), 0, st, s.counter_dev, (int32_t)w, s.leader_dev, leader_out);
      HIP_TRY(ctx, hipGetLastError());
    }
    if (leader_first) ctx->last_dom_workers = 1;
    ctx->last_short = 1;
    ctx->last_one_launch = 0;
    return small_step(ctx, gt, rt, w, n, k, mode == ARTOPK_VAR ? 1 : mode == ARTOPK_VAR_G ? 2 : 0,
                      leader_first ? leader_host : -1, leader_out, var_out, idx_out, vals_out, sum_out, update_out);
  }

  if (leader_first) {
    // The leader is known up front: run its pass and the selection first, then
    // stream over the other workers once, gathering and zeroing on the way.
    const int L = leader_host;
    ctx->lvl1_a = 2;
    ctx->lvl1_b = 3;
    float* vals = vals_out ? vals_out : s.vals;
    const float* g1[1] = {g[L]};
    const float* r1[1] = {residual[L]};
    const PtrTable g1t = make_table(g1, 1), r1t = make_table(r1, 1);
    prof_begin(ctx);
    prof_mark(ctx, 0);
    const bool tiles = segmented ? by_tiles : gp.tiles;
    if ((rc = enqueue_clear(ctx, *pl, segmented ? 0 : 1, L, leader_out, tiles))) return rc;
    ctx->last_guessed = gp.on ? 1 : 0;
    ctx->last_dom_workers = w > 1 ? w - 1 : 1;
    if (gp.on && !tiles) enqueue_guess(ctx, gp, g1t, r1t, 1);
    if (tiles) {
      if ((rc = enqueue_tiles(ctx, *pl, rt, n, idx_out, vals + (size_t)L * (size_t)k, gp, g[L], residual[L], true))) return rc;
    } else {
      if (gp.on) {
        launch_pass_mark(ctx, 0, 1, g1t, r1t, n, geom.chunk_elems);
      } else if (segmented) {
        if (g_type == ARTOPK_G_BF16)
          launch_pass_seg<kGBF16>(ctx, *pl, rt, n, g[L], residual[L]);
        else if (g_type == ARTOPK_G_F16)
          launch_pass_seg<kGF16>(ctx, *pl, rt, n, g[L], residual[L]);
        else
          launch_pass_seg<kGF32>(ctx, *pl, rt, n, g[L], residual[L]);
        HIP_TRY(ctx, hipGetLastError());
      } else {
        launch_pass_a(ctx, 0, 1, dim3(geom.nchunks, 1), g1t, r1t, n, geom, 0);
      }
      prof_mark(ctx, 1);
      // The leader's residual is zeroed inside the selection: its kernels have the kept values in
      // registers (level-1 compaction) or write the kept indices anyway (final list pass).
      if ((rc = enqueue_select(ctx, *pl, rt, n, idx_out, !segmented, 0, vals + (size_t)L * (size_t)k, nullptr, gp.on,
                               residual[L], 0, nullptr, segmented)))
        return rc;
    }
    prof_mark(ctx, 2);
    const int rest = (int)w - 1;
    if (!tiles || !pl->tiles_aligned) enqueue_tile_starts(ctx, idx_out, n, k);  // (else k_tiles_out has left them)
    prof_dom(ctx, false);
    if (rest > 0) {
      launch_pass_rest(ctx, gt, rt, (int)w, L, n, idx_out, k, vals);
    }
    prof_dom(ctx, true);
    prof_mark(ctx, 3);
    if (update_out && k * 128 <= n) {
      // few kept entries: the ordered sums and the dense update in one pass over the tiles, whose bounds
      // in idx are there already (138 M elements, one in a thousand kept: 96 us against 104 + 4; one in a
      // hundred: 133 against 116 + 5, the owner threads' loads of the rows' entries take over)
      hipLaunchKernelGGL((k_sum_update<kPassRestThreads, kPassRestU>), dim3(pass_blocks(n)), dim3(kPassRestThreads),
                         0, st, vals, (int)w, n, idx_out, k, s.tile_start, sum_out, update_out, s.err_dev);
      HIP_TRY(ctx, hipGetLastError());
    } else {
      hipLaunchKernelGGL(k_sum_rows, dim3((int)((k + 1023) / 1024)), dim3(256), 0, st, vals, (int)w, k, sum_out);
      HIP_TRY(ctx, hipGetLastError());
      if (update_out && (rc = enqueue_update_fill(ctx, update_out, n, idx_out, sum_out, k, true))) return rc;
    }
    prof_mark(ctx, 4);
    return ARTOPK_OK;
  }

  ctx->lvl1_a = 0;
  ctx->lvl1_b = 1;
  prof_begin(ctx);
  prof_mark(ctx, 0);
  // the flat select reuses the histograms pass A builds; segments build their own afterwards
  if ((rc = enqueue_clear(ctx, *pl, segmented ? 0 : (device_leader ? (int)w : 1), -1, nullptr, by_tiles))) return rc;
  int slot_by_leader = 0;
  LeaderArgs leader_args{};
  const bool marking = gp.on && device_leader;
  if (mode == ARTOPK_STAR_COUNTER) {
    // every worker's pass prepares the selection, as under the variance rules, and the selection
    // kernels read the leader word that the counter kernel leaves
    hipLaunchKernelGGL(k_counter_leader, dim3(1), dim3(64), 0, st, s.counter_dev, (int32_t)w, s.leader_dev, leader_out);
    HIP_TRY(ctx, hipGetLastError());
    ctx->last_guessed = marking ? 1 : 0;
    if (marking) enqueue_guess(ctx, gp, gt, rt, (int)w);
    prof_dom(ctx, false);
    if (seg_stride) {
      launch_pass_plain(ctx, 0, (int)w, gt, rt, n);
    } else if (segmented) {
      launch_pass_a(ctx, 0, 0, grid, gt, rt, n, geom, -1);
    } else if (marking) {
      launch_pass_mark(ctx, 0, (int)w, gt, rt, n, geom.chunk_elems);
      slot_by_leader = 1;
    } else {
      launch_pass_a(ctx, 0, 2, grid, gt, rt, n, geom, -1, by_tile);
      slot_by_leader = 1;
    }
    prof_dom(ctx, true);
    prof_mark(ctx, 1);
  } else if (mode == ARTOPK_VAR || mode == ARTOPK_VAR_G) {
    const int stats = mode == ARTOPK_VAR_G ? 2 : 1;  // variance of the raw gradient, or of g + residual
    if (segmented) {
      prof_dom(ctx, false);
      if (seg_stride)
        launch_pass_plain(ctx, stats, (int)w, gt, rt, n);
      else
        launch_pass_a(ctx, stats, 0, grid, gt, rt, n, geom, -1);
    } else {
      ctx->last_guessed = gp.on ? 1 : 0;
      if (gp.on) enqueue_guess(ctx, gp, gt, rt, (int)w);
      prof_dom(ctx, false);
      if (gp.on) {
        launch_pass_mark(ctx, stats, (int)w, gt, rt, n, geom.chunk_elems);
      } else {
        launch_pass_a(ctx, stats, 2, grid, gt, rt, n, geom, -1, by_tile);
      }
      slot_by_leader = 1;
    }
    prof_dom(ctx, true);
    prof_mark(ctx, 1);
    if (segmented) {  // the segment histograms are built on the leader's vector, so it is needed now
      hipLaunchKernelGGL(k_leader, dim3(1), dim3(1024), 0, st, s.partials, (int)w,
                         seg_stride ? pass_blocks(n) : (int)geom.nchunks, n, s.var_scratch, var_out, s.leader_dev,
                         leader_out);
    } else {          // otherwise the selection's first kernel takes the leader itself
      leader_args.partials = s.partials;
      leader_args.w_count = (int)w;
      leader_args.nblk = marking ? pass_blocks(n) : pass_nblk;
      leader_args.n = n;
      leader_args.var_scratch = s.var_scratch;
      leader_args.var_out = var_out;
      leader_args.leader_dev = s.leader_dev;
      leader_args.leader_out = leader_out;
    }
  } else {
    prof_dom(ctx, false);
    if (seg_stride)
      launch_pass_plain(ctx, 0, (int)w, gt, rt, n);
    else
      launch_pass_a(ctx, 0, segmented ? 0 : 1, grid, gt, rt, n, geom, leader_host, by_tile);
    prof_dom(ctx, true);
    prof_mark(ctx, 1);
    hipLaunchKernelGGL(k_set_leader, dim3(1), dim3(64), 0, st, (int32_t)leader_host, s.leader_dev, leader_out);
  }
  HIP_TRY(ctx, hipGetLastError());

  rc = by_tiles ? enqueue_tiles(ctx, *pl, rt, n, idx_out, nullptr, gp, nullptr, nullptr, false)
                : enqueue_select(ctx, *pl, rt, n, idx_out, !segmented, slot_by_leader, nullptr,
                                 leader_args.partials ? &leader_args : nullptr, marking);
  if (rc) return rc;
  prof_mark(ctx, 2);
  if ((rc = enqueue_gather(ctx, rt, w, n, idx_out, k, vals_out, sum_out, true))) return rc;
  prof_mark(ctx, 3);
  if (update_out && (rc = enqueue_update_fill(ctx, update_out, n, idx_out, sum_out, k))) return rc;
  prof_mark(ctx, 4);
  return ARTOPK_OK;
}

}  // namespace

int artopk_set_step_counter(artopk_ctx* ctx, uint64_t value) {
  if (!ctx) return fail(nullptr, ARTOPK_EINVAL, "artopk_set_step_counter: ctx is NULL");
  hipLaunchKernelGGL(k_set_counter, dim3(1), dim3(64), 0, ctx->stream, ctx->s.counter_dev, value);
  HIP_TRY(ctx, hipGetLastError());
  return ARTOPK_OK;
}

int artopk_step(artopk_ctx* ctx, const float* const* g, float* const* residual, int32_t w, int64_t n,
                int32_t nseg, const int64_t* seg_off, const int64_t* seg_k, int64_t k, int32_t mode,
                uint64_t step, int32_t fixed_leader, int32_t* leader_out, double* var_out, int32_t* idx_out,
                float* vals_out, float* sum_out, float* update_out) {
  return step_impl(ctx, g, ARTOPK_G_F32, residual, w, n, nseg, seg_off, seg_k, k, mode, step, fixed_leader,
                   leader_out, var_out, idx_out, vals_out, sum_out, update_out);
}

int artopk_step_g16(artopk_ctx* ctx, const void* const* g, int32_t g_type, float* const* residual, int32_t w,
                    int64_t n, int32_t nseg, const int64_t* seg_off, const int64_t* seg_k, int64_t k,
                    int32_t mode, uint64_t step, int32_t fixed_leader, int32_t* leader_out, double* var_out,
                    int32_t* idx_out, float* vals_out, float* sum_out, float* update_out) {
  if (ctx && g_type != ARTOPK_G_BF16 && g_type != ARTOPK_G_F16)
    return fail(ctx, ARTOPK_EINVAL, "artopk_step_g16 takes ARTOPK_G_BF16 or ARTOPK_G_F16 gradients");
  return step_impl(ctx, reinterpret_cast<const float* const*>(g), g_type, residual, w, n, nseg, seg_off, seg_k, k,
                   mode, step, fixed_leader, leader_out, var_out, idx_out, vals_out, sum_out, update_out);
}

}  // extern "C"

#ifdef ARTOPK_HELD_BLOCKS
// For tests of how blocks take on others' work: sets HeldBlocks and says how many units were taken on since the last call.
extern "C" int artopk_held_blocks(uint32_t ticks, uint32_t looks, uint32_t* helped_out) {
  HeldBlocks h{};
  if (hipDeviceSynchronize() != hipSuccess || hipMemcpyFromSymbol(&h, HIP_SYMBOL(held_blocks), sizeof(h)) != hipSuccess)
    return ARTOPK_EHIP;
  *helped_out = h.helped;
  h = HeldBlocks{ticks, looks, 0u};
  return hipMemcpyToSymbol(HIP_SYMBOL(held_blocks), &h, sizeof(h)) == hipSuccess ? ARTOPK_OK : ARTOPK_EHIP;
}
#endif
