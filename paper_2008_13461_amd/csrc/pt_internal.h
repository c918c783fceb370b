// Internal declarations shared by the HIP sources of the pixel-track library.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "../../include/pixeltrack.h"

namespace pt {

constexpr int kWave = 64;
constexpr int kLayers = PT_N_LAYERS;
constexpr int kMaxPairs = PT_MAX_PAIRS;
constexpr int kMaxHits = PT_MAX_HITS;
constexpr int kMaxPairsPerLayer = 8;
constexpr int kRzBuckets = 128;  // direction buckets of the windowed R-Z search, at most

// Constants the kernels use, derived once on the host from pt_config
// (see the expressions documented in pixeltrack.h).
struct DevCfg {
  // doublets
  double tan_dphi[kMaxPairs];
  double zlo[kMaxPairs];
  double zhi[kMaxPairs];
  double z0_max;
  double kappa_max2;
  uint32_t cut_mask;
  int32_t n_pairs;
  int32_t n_bins;                       // azimuth bins per layer
  int32_t bin_shift;                    // log2(n_bins) when a power of two, else -1
  float bin_scale;                      // n_bins / (2 pi)
  int32_t pair_inner[kMaxPairs];
  int32_t pair_outer[kMaxPairs];
  int32_t pair_wbins[kMaxPairs];        // half window in bins (>= n_bins/2: whole layer)
  int32_t inner_pairs[kLayers][kMaxPairsPerLayer];  // pairs whose inner layer is l, -1 padded
  int32_t n_inner_pairs[kLayers];
  // links
  double theta2_barrel, theta2_endcap;
  uint32_t endcap_pairs;  // bit p set when the outer layer of pair p is an end-cap layer
  int32_t rz_buckets;  // direction buckets of the windowed R-Z search (0: every pair is tested)
  double rmax_bpix1, rmax_other;
  uint8_t layer_barrel[kLayers];
  // n-tuplets
  uint32_t root_always_mask, root_if_free_mask;
  int32_t min_hits, max_hits;
  // fit
  double K;          // 0.299792458 B / 100
  double x_over_x0, highland_a, highland_b;
  double VT, VZ_barrel, VR_disk, p_cap;
  double f64_threshold;
  int32_t n_modules;
  int32_t block_doublets;
  // vertices
  int32_t vtx_min_hits, vtx_kmeans_iter;
  double vtx_pt_min, vtx_err_max, vtx_dz_cut, vtx_chi2_max, vtx_split_chi2_ndf, vtx_pt_cap;
  // Fishbone (0: off)
  double fishbone_theta2;
  // adjoint: grad_hits rows are written by one track each
  int32_t exclusive_hits;
};

bool derive_config(const pt_config& c, DevCfg* d);

// ---------------------------------------------------------------------------
// Workspace carving: every region 256-byte aligned.
struct Carver {
  char* base;
  size_t off = 0;
  explicit Carver(void* p) : base(static_cast<char*>(p)) {}
  template <class T>
  T* take(size_t n) {
    off = (off + 255) & ~size_t(255);
    T* p = reinterpret_cast<T*>(base + off);
    off += n * sizeof(T);
    return p;
  }
};

// Workspace needed by each call (bytes); the public size is their maximum.
size_t ws_doublets(int n_hits, int n_events, int n_bins, int raw_cells);  // raw_cells: capacity when the Fishbone is on, else 0
size_t ws_links(int n_hits, int cells_cap);
size_t ws_ntuplets(int cells_cap, int tuplets_cap);
size_t ws_fit(int n_max, int n_modules);
size_t ws_ambiguity(int n_hits, int cells_cap, int n_max);
// The Fishbone filters the cells as the doublet step finds them, in the
// workspace, into the output: carve_raw_cells carves them (the rest of
// `cells` is shared), launch_fishbone takes its scratch behind them.
size_t ws_fishbone(int n_hits, int cells_cap);
pt_cells carve_raw_cells(Carver& c, const pt_cells& cells, int cells_cap);
pt_err launch_fishbone(const pt_hits& h, const DevCfg& k, const pt_cells& raw, pt_cells& cells, Carver c,
                       hipStream_t s);
// Host-side set-up of the Fishbone's launch shapes (device queries), done
// before a plan captures its graph.
void fishbone_prepare();

// The index of the stored cells by outer hit (links.hip): hit h's cells are
// the entries ent[f .. f + k) (cell, inner hit with bit 31 set when on
// BPix1) of its segments (f, k) = seg[seg_first[h] .. seg_first[h + 1]).
// The cells must not have overflowed their capacity.
struct OuterIndex {
  const int2* ent;
  const int2* seg;
  const int32_t* seg_first;
};
size_t ws_outer_index(int n_hits, int cells_cap);
pt_err build_outer_index(const pt_hits& h, const pt_cells& cells, Carver& c, OuterIndex& out, hipStream_t s);
size_t ws_vertices(int n_events, int n_max);

// Device-wide exclusive scans, one kernel each: every work-group scans a tile
// of kTileItems consecutive values, kScanItems per thread, and takes the sum of
// the tiles before its own from their states (see tile_before below).  state
// holds scan_state_words(n) words, zero before the kernel runs; a scan of one
// tile does not use it.
constexpr int kTileThreads = 256;
constexpr int kScanItems = 16;
constexpr int kTileItems = kTileThreads * kScanItems;
constexpr size_t tiles_of(int64_t n, int64_t tile) { return n > 0 ? static_cast<size_t>((n + tile - 1) / tile) : 1; }
constexpr size_t scan_state_words(int64_t n) { return tiles_of(n, kTileItems); }
// Above this many cells (the capacity) a listing takes its tiles' offsets from a
// pass over their sums instead: the chain of states (8 ns a tile) is then longer
// than the pass.  In one kernel and with the pass, 1, 2, 4, 8 and 64 events of
// 200 vertices (740, 1470, 2940, 5860 and 46 700 tiles): pt_link_cells 133, 214,
// 416, 796, 5713 and 134, 211, 406, 759, 5314 us, pt_find_ntuplets 84, 107, 168,
// 272, 1704 and 89, 105, 157, 243, 1352 us.  The line, 4096 tiles of capacity,
// lies above the crossing, which is near 1000 tiles of cells.
constexpr int64_t kLargeItems = int64_t(1) << 24;
// dst[i] = src[0] + .. + src[i-1] over the first m = min(*n_dev, n) values,
// n_dev a device count (n when null), dst[m] the total, which also goes to
// *total when given, with `flag` set in the status when it exceeds cap.  src
// and dst must not overlap.  The sums saturate (count_add below).
struct ScanTotal {
  int32_t* total = nullptr;
  int32_t cap = 0x7fffffff;
  uint32_t flag = 0;
  uint32_t* status = nullptr;
};
hipError_t exclusive_scan(const int32_t* src, int32_t* dst, int64_t n, const int32_t* n_dev, const ScanTotal& t,
                          uint64_t* state, hipStream_t s);
// Sums of the tiles of kTileItems of the first min(*n_dev, n) values (0 past
// them), one per tile of n.
hipError_t tile_sums(const int32_t* src, int64_t n, const int32_t* n_dev, int32_t* sums, hipStream_t s);

// Fill helpers (graph-safe: kernels, not hipMemsetAsync).
hipError_t fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t s);
hipError_t fill_u8(uint8_t* p, uint8_t v, int64_t n, hipStream_t s);

// grid size for grid-stride loops over n items
inline int grid_for(int64_t n, int block, int max_blocks = 65536) {
  int64_t g = (n + block - 1) / block;
  if (g < 1) g = 1;
  if (g > max_blocks) g = max_blocks;
  return static_cast<int>(g);
}

// Kernel timing hooks (no-ops unless pt_timing_enable(1) and not capturing).
void* timing_begin(hipStream_t s);
void timing_end(void* token, const char* name, hipStream_t s);
extern thread_local bool g_capturing;
extern thread_local bool g_no_timing;  // set by entry points that must not create events

// Device errors: the HIP error behind a PT_ERR_DEVICE is kept per host thread
// (pt_last_device_error).  Entry points clear the thread's HIP error state
// before they launch, so that an error another caller left there (an event
// query's hipErrorNotReady, say) is not taken for one of theirs.
pt_err device_error(hipError_t e);
inline void clear_stale_error() { (void)hipGetLastError(); }

#define PT_HIP_CHECK(expr)                                   \
  do {                                                       \
    const hipError_t pt_e_ = (expr);                         \
    if (pt_e_ != hipSuccess) return ::pt::device_error(pt_e_); \
  } while (0)

#define PT_LAUNCH_CHECK() PT_HIP_CHECK(hipGetLastError())

// ---------------------------------------------------------------------------
// device helpers

// Four values of the input type in one vector (one load).
template <class T>
struct Vec4Of;
template <>
struct Vec4Of<float> { using type = float4; };
template <>
struct Vec4Of<double> { using type = double4; };
template <class T>
using Vec4 = typename Vec4Of<T>::type;

__device__ inline void status_flag(uint32_t* st, uint32_t bit) {
  if (st) atomicOr(st + PT_ST_FLAGS, bit);
}
__device__ inline void status_add(uint32_t* st, int word, uint32_t v) {
  if (st && v) atomicAdd(st + word, v);
}

// status_add summed over the wavefront first: one atomic per wavefront.  All
// lanes of the wavefront must call it.
// Returns the wavefront's total.
__device__ inline uint32_t wave_status_add(uint32_t* st, int word, uint32_t v) {
#pragma unroll
  for (int d = kWave / 2; d > 0; d >>= 1) v += __shfl_xor(v, d, kWave);
  if (__lane_id() == 0) status_add(st, word, v);
  return v;
}

// Sum and inclusive prefix sum over the wavefront; all lanes must call them.
__device__ inline int wave_sum(int v) {
#pragma unroll
  for (int d = kWave / 2; d > 0; d >>= 1) v += __shfl_xor(v, d, kWave);
  return v;
}
// The scans move their partial results with DPP (within rows of 16 lanes,
// then across rows) instead of through the LDS permute unit, whose latency
// six dependent steps would pay six times.  A lane without a source combines
// with `none`.
template <class F>
__device__ __forceinline__ int wave_scan_with(int v, int none, F f) {
  v = f(v, __builtin_amdgcn_update_dpp(none, v, 0x111, 0xf, 0xf, false));  // row_shr:1, 2, 4, 8
  v = f(v, __builtin_amdgcn_update_dpp(none, v, 0x112, 0xf, 0xf, false));
  v = f(v, __builtin_amdgcn_update_dpp(none, v, 0x114, 0xf, 0xf, false));
  v = f(v, __builtin_amdgcn_update_dpp(none, v, 0x118, 0xf, 0xf, false));
  v = f(v, __builtin_amdgcn_update_dpp(none, v, 0x142, 0xa, 0xf, false));  // row_bcast:15 into rows 1 and 3
  v = f(v, __builtin_amdgcn_update_dpp(none, v, 0x143, 0xc, 0xf, false));  // row_bcast:31 into rows 2 and 3
  return v;
}
__device__ __forceinline__ int wave_incl_scan(int v) {
  return wave_scan_with(v, 0, [](int a, int b) { return a + b; });
}
__device__ __forceinline__ int wave_max_scan(int v) {
  return wave_scan_with(v, -0x7fffffff - 1, [](int a, int b) { return max(a, b); });
}

// Counts of cells, links and rows may exceed 32 bits (a batch with wide cuts has
// billions of candidates): their sums saturate at kMaxCount, so that a position
// past it lies past every capacity, which is at most kMaxItems, instead of
// wrapping round to a place before the buffers.  Counts are not negative, so
// the signed saturating add (one instruction) is associative on them.
constexpr int32_t kMaxCount = 0x7fffffff;
// What is counted as capacity: below kMaxCount, so that a saturated total always
// exceeds it, by more than the step of any grid-stride loop over it.
constexpr int32_t kMaxItems = kMaxCount - (1 << 25);
inline int32_t capacity(int32_t cap) { return cap < kMaxItems ? cap : kMaxItems; }
__device__ __forceinline__ int32_t count_add(int32_t a, int32_t b) { return __builtin_elementwise_add_sat(a, b); }
__device__ __forceinline__ int32_t wave_count_scan(int32_t v) {
  return wave_scan_with(v, 0, [](int a, int b) { return count_add(a, b); });
}
__device__ inline int32_t wave_count_sum(int32_t v) { return __builtin_amdgcn_readlane(wave_count_scan(v), kWave - 1); }
// The exclusive prefix, from the inclusive one (a difference would not be the
// prefix of a saturated sum).
__device__ inline int32_t wave_before(int32_t incl) {
  const int32_t v = __shfl_up(incl, 1, kWave);
  return __lane_id() > 0 ? v : 0;
}

// Minimum over the wavefront, the same in every lane.
__device__ __forceinline__ float wave_min(float v) {
  const int r = wave_scan_with(__float_as_int(v), __float_as_int(__builtin_inff()), [](int a, int b) {
    return __float_as_int(fminf(__int_as_float(a), __int_as_float(b)));
  });
  return __int_as_float(__builtin_amdgcn_readlane(r, kWave - 1));
}

// ---------------------------------------------------------------------------
// Prefixes over the tiles of one kernel (decoupled look-back), tile i the
// work-group i.  The state of
// a tile is a value in the low word, and above it 0 (not there yet), kTileSum
// (the tile's own sum) or kTilePrefix (the sum up to and including it).  Value
// and flag are one atomic, so no other memory is ordered by it.  A work-group
// waits for the tiles before its own a bounded number of polls and then sums
// the missing tile itself, from the input (which no tile overwrites): every
// wait ends, in whatever order the work-groups are started.  (A ticket per
// tile, taken in the order the work-groups start, orders them too, but one
// counter hands out a ticket every 11 ns: 15 us for the tiles of one pileup-200
// event.)
constexpr uint64_t kTileSum = uint64_t(1) << 32, kTilePrefix = uint64_t(2) << 32;
#ifndef PT_TILE_POLLS
#define PT_TILE_POLLS 256  // negative (a test build): no state is read, every work-group sums for itself
#endif
constexpr int kPolls = PT_TILE_POLLS;

// The sum of the tiles before `tile`, whose own sum is given; called by one
// wavefront.  sum_of(i), called by the whole wavefront, is the sum of tile i.
// Lanes look back 64 tiles at a time to the last one whose prefix is known, the
// loads of kLookBack such steps in flight together: a state comes from beyond
// the XCD's own L2, and the tiles of every resident work-group lie between a
// tile and the last known prefix.
constexpr int kLookBack = 8;
template <class F>
__device__ inline int32_t tile_before(uint64_t* state, int tile, int32_t sum, F sum_of) {
  const int lane = __lane_id();
  auto load = [&](int i) {
    if (i < 0) return kTilePrefix;
    return kPolls < 0 ? uint64_t(0) : __hip_atomic_load(state + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  if (lane == 0)
    __hip_atomic_store(state + tile, (tile == 0 ? kTilePrefix : kTileSum) | static_cast<uint32_t>(sum),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  int32_t before = 0;
  bool done = tile == 0;
  for (int at = tile - 1; !done; at -= kLookBack * kWave) {
    uint64_t v[kLookBack];
#pragma unroll
    for (int k = 0; k < kLookBack; ++k) v[k] = load(at - k * kWave - lane);
#pragma unroll
    for (int k = 0; k < kLookBack; ++k) {
      if (done) continue;
      const int first = at - k * kWave;  // lane 0's tile
      uint64_t known;                    // lanes whose tile's prefix is known
      for (int polls = 0;; ++polls) {
        known = __ballot(v[k] >= kTilePrefix);
        const uint64_t wanted = known ? (known & (~known + 1)) * 2 - 1 : ~uint64_t(0);  // up to the nearest
        const uint64_t missing = __ballot(v[k] == 0) & wanted;
        if (!missing) break;
        if (polls < kPolls) {
          if (v[k] == 0) v[k] = load(first - lane);
        } else {
          const int l = __builtin_ctzll(missing);
          const int32_t x = sum_of(first - l);
          if (lane == l) v[k] = kTileSum | static_cast<uint32_t>(x);
        }
      }
      const int stop = known ? __builtin_ctzll(known) : kWave;
      before = count_add(before, wave_count_sum(lane <= stop ? static_cast<int32_t>(static_cast<uint32_t>(v[k])) : 0));
      done = known != 0;
    }
  }
  if (lane == 0 && tile > 0)
    __hip_atomic_store(state + tile, kTilePrefix | static_cast<uint32_t>(count_add(before, sum)),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return before;
}

// Exclusive prefix of v over the work-group (kTileThreads) and, with a state,
// the tiles before its own; *end receives the sum up to and including the
// tile, s_wave[0] the sum before it.  s_wave holds kTileThreads / kWave + 1 words.
// The sums saturate, sum_of's as well (a sum over the wavefront: wave_count_sum).
template <class F>
__device__ inline int32_t tile_exclusive(int32_t v, uint64_t* state, int tile, int32_t* s_wave, int32_t* end, F sum_of) {
  constexpr int kWaves = kTileThreads / kWave;
  const int lane = __lane_id(), wave = static_cast<int>(threadIdx.x) / kWave;
  const int32_t incl = wave_count_scan(v);
  if (lane == kWave - 1) s_wave[wave] = incl;
  __syncthreads();
  if (wave == 0) {
    const int32_t wi = wave_count_scan(lane < kWaves ? s_wave[lane] : 0);
    const int32_t sum = __builtin_amdgcn_readlane(wi, kWaves - 1);
    const int32_t before = state ? tile_before(state, tile, sum, sum_of) : 0;
    const int32_t first = count_add(before, wave_before(wi));
    if (lane < kWaves) s_wave[lane] = first;
    if (lane == 0) s_wave[kWaves] = count_add(before, sum);
  }
  __syncthreads();
  *end = s_wave[kWaves];
  return count_add(s_wave[wave], wave_before(incl));
}
__device__ inline int32_t block_exclusive(int32_t v, int32_t* s_wave, int32_t* total) {
  return tile_exclusive(v, nullptr, 0, s_wave, total, [](int) { return 0; });
}

// Positions of a tile of four runs of flags, c[i] the number of set flags of
// this thread's group in run i (the groups of a run in thread order): pos[i]
// is the number of set flags before c[i]'s first, in the tile and (with a
// state) those before it, *end the number up to the tile's end.  s_wave holds
// 2 kTileThreads / kWave + 3 words.  The sum of a run fits 15 bits.
template <class F>
__device__ inline void tile_positions(const int (&c)[4], uint64_t* state, int tile, int32_t* s_wave, int (&pos)[4],
                                      int32_t* end, F sum_of) {
  constexpr int kWaves = kTileThreads / kWave;
  const int lane = __lane_id(), wave = static_cast<int>(threadIdx.x) / kWave;
  const int a = c[0] | c[1] << 16, b = c[2] | c[3] << 16;
  const int ia = wave_incl_scan(a), ib = wave_incl_scan(b);
  if (lane == kWave - 1) {
    s_wave[wave] = ia;
    s_wave[kWaves + wave] = ib;
  }
  __syncthreads();
  if (wave == 0) {
    const int wa = lane < kWaves ? s_wave[lane] : 0, wb = lane < kWaves ? s_wave[kWaves + lane] : 0;
    const int sa = wave_incl_scan(wa), sb = wave_incl_scan(wb);
    const int ta = __builtin_amdgcn_readlane(sa, kWaves - 1), tb = __builtin_amdgcn_readlane(sb, kWaves - 1);
    const int sum = (ta & 0xFFFF) + (ta >> 16) + (tb & 0xFFFF) + (tb >> 16);
    const int32_t before = state ? tile_before(state, tile, sum, sum_of) : 0;
    if (lane < kWaves) {  // the wavefronts' first positions within each run
      s_wave[lane] = sa - wa;
      s_wave[kWaves + lane] = sb - wb;
    }
    if (lane == 0) {
      s_wave[2 * kWaves] = before;
      s_wave[2 * kWaves + 1] = ta;
      s_wave[2 * kWaves + 2] = tb;
    }
  }
  __syncthreads();
  const int ta = s_wave[2 * kWaves + 1], tb = s_wave[2 * kWaves + 2];
  const int ea = s_wave[wave] + ia - a, eb = s_wave[kWaves + wave] + ib - b;
  const int b0 = s_wave[2 * kWaves], b1 = b0 + (ta & 0xFFFF), b2 = b1 + (ta >> 16), b3 = b2 + (tb & 0xFFFF);
  pos[0] = b0 + (ea & 0xFFFF);
  pos[1] = b1 + (ea >> 16);
  pos[2] = b2 + (eb & 0xFFFF);
  pos[3] = b3 + (eb >> 16);
  *end = b3 + (tb >> 16);
}

// kScanItems consecutive values of a thread, from index `base` of n (16-byte
// vectors where they lie below n, when VEC); values past n are 0.
template <bool VEC>
__device__ inline void load_items(const int32_t* src, int64_t base, int64_t n, int32_t (&v)[kScanItems]) {
#pragma unroll
  for (int i = 0; i < kScanItems; i += 4) {
    if (VEC && base + i + 4 <= n) {
      const int4 q = *reinterpret_cast<const int4*>(src + base + i);
      v[i] = q.x;
      v[i + 1] = q.y;
      v[i + 2] = q.z;
      v[i + 3] = q.w;
    } else {
#pragma unroll
      for (int k = i; k < i + 4; ++k) v[k] = base + k < n ? src[base + k] : 0;
    }
  }
}
template <bool VEC>
__device__ inline void store_items(int32_t* dst, int64_t base, int64_t n, const int32_t (&v)[kScanItems]) {
#pragma unroll
  for (int i = 0; i < kScanItems; i += 4) {
    if (VEC && base + i + 4 <= n) {
      *reinterpret_cast<int4*>(dst + base + i) = make_int4(v[i], v[i + 1], v[i + 2], v[i + 3]);
    } else {
#pragma unroll
      for (int k = i; k < i + 4; ++k)
        if (base + k < n) dst[base + k] = v[k];
    }
  }
}
__host__ __device__ inline bool aligned16(const void* p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; }

// Number of set bits of a wave mask below this lane.
__device__ inline int lane_prefix(uint64_t mask) {
  return static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                                    __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u)));
}

// Work-group dispatch places consecutive work-group ids on different XCDs
// (round robin over kXcds), each with its own L2.  xcd_block(b, m) renumbers
// the work-groups of a 1-D grid so that each XCD takes runs of m.run consecutive
// logical ids: neighbouring work-groups, which read and write neighbouring
// memory, then share an L2 and complete its cache lines there.  The grid is
// whole rounds of kXcds runs (xcd_grid), so that there is no last round to tell
// apart: the wavefronts issue more scalar than vector instructions before the
// first candidate.
constexpr int kXcds = 8;
struct XcdRuns {
  int32_t run;
  int32_t shift;  // log2 of the ids of a round, 31 for a single round
};
inline XcdRuns xcd_runs(int shift) { return {(1 << shift) / kXcds, shift}; }
inline XcdRuns xcd_ranges(int64_t nb) { return {static_cast<int32_t>((nb + kXcds - 1) / kXcds), 31}; }
inline unsigned xcd_grid(int64_t nb, const XcdRuns& m) {
  const int64_t round = static_cast<int64_t>(m.run) * kXcds;
  return static_cast<unsigned>((nb + round - 1) / round * round);
}
__device__ inline int xcd_block(unsigned b, const XcdRuns& m) {
  const unsigned first = b >> m.shift << m.shift;
  return static_cast<int>(first + b % kXcds * m.run + (b - first) / kXcds);
}

// Orders the LDS traffic of one wavefront (its lanes run in lockstep, so a
// compiler barrier is all that is needed between a write and a read by
// another lane).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace pt
