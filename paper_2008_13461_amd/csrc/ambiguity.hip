// Ambiguity resolution among fitted tracks (paper section 3.5).
//
// Tracks sharing a hit doublet (a cell) are ambiguous and only the one with
// the smallest chi^2 stays; then, among the 3-hit tracks that stayed, tracks
// sharing a hit are ambiguous and only the one with the smallest transverse
// impact parameter |d0| stays.  Equal values keep both.  Tracks whose fit
// failed (non-finite chi^2) take no part and are not selected.
//
// Both rules are a minimum per key (cell, then hit) followed by a test of
// each track against the minima of its keys, as the duplicate removal of the
// n-tuplet search does with its maximum per cell.  Values are compared as
// the bit patterns of their magnitudes (for non-negative numbers the unsigned
// order of the bits is the numeric order), so one atomicMin of the outputs'
// width per (track, key) takes each minimum.  The minima are reset first: for
// the keys the tracks visit, so that the cost follows the number of tracks,
// or all of them in one stream when that is cheaper.  Selected tracks are
// listed in track order (flags, a scan, a scatter).
#include <algorithm>

#include "pt_internal.h"

namespace pt {
namespace {

constexpr int kBlock = 256;

struct AmbArgs {
  const int32_t* hits;   // rows [cap][kMaxHits]
  const int32_t* cells;  // rows [cap][kMaxHits - 1]
  const uint8_t* n;      // [cap]
  const int32_t* kept;   // track i is row kept[i] (row i when null)
  const int32_t* count;  // number of tracks (device)
  int32_t n_max;
  const void* chi2;      // [n_max], double when dbl else float
  const void* params;    // [n_max][5]
  int32_t n_hits, n_cells;
  void* best_cell;       // [n_cells] keys (Key<T>)
  void* best_hit;        // [n_hits]
  int32_t* flag;         // [n_max]: 0 dropped, 1 kept, 2 triplet kept by the chi2 rule (pass 1)
  int32_t* pos;          // [n_max + 1]
  uint64_t* state;       // of the scan of the flags, cleared with the minima
  int32_t state_words;
};

__device__ inline int n_tracks(const AmbArgs& a) { return min(*a.count, a.n_max); }

// Order key of a magnitude: the bits of |v|, T the type of the fit's outputs.
template <class T>
using Key = typename std::conditional<sizeof(T) == 4, unsigned int, unsigned long long>::type;
__device__ inline unsigned int key_of(float v) { return __float_as_uint(fabsf(v)); }
__device__ inline unsigned long long key_of(double v) {
  return static_cast<unsigned long long>(__double_as_longlong(fabs(v)));
}


// A track takes part when its fit succeeded and its row indexes valid cells
// and hits.
template <class T>
__device__ inline bool candidate(const AmbArgs& a, int i, int& row, int& nh) {
  row = a.kept ? a.kept[i] : i;
  nh = a.n[row];
  if (nh < 2 || nh > kMaxHits) return false;
  if (!isfinite(static_cast<const T*>(a.chi2)[i])) return false;
  const int32_t* C = a.cells + static_cast<int64_t>(row) * (kMaxHits - 1);
  for (int d = 0; d < nh - 1; ++d)
    if (C[d] < 0 || C[d] >= a.n_cells) return false;
  if (nh == 3) {
    const int32_t* H = a.hits + static_cast<int64_t>(row) * kMaxHits;
    for (int d = 0; d < 3; ++d)
      if (H[d] < 0 || H[d] >= a.n_hits) return false;
  }
  return true;
}

// Keys per track up to which all minima are reset in one stream (1 ps a key)
// instead of those that the tracks visit (50 ps a track): 9.2 million triplets
// and 40 million cells 463 -> 40 us.
constexpr int kStreamKeys = 16;

template <class T>
__global__ void __launch_bounds__(kBlock) k_amb_reset(AmbArgs a) {
  constexpr Key<T> kNone = ~Key<T>(0);
  const int n = n_tracks(a);
  const int first = blockIdx.x * kBlock + threadIdx.x, step = gridDim.x * kBlock;
  for (int i = first; i < a.state_words; i += step) a.state[i] = 0;
  Key<T>* cell = static_cast<Key<T>*>(a.best_cell);
  Key<T>* hit = static_cast<Key<T>*>(a.best_hit);
  if (a.n_cells / kStreamKeys <= n && a.n_hits / kStreamKeys <= n) {
    constexpr int kVec = sizeof(uint4) / sizeof(Key<T>);
    uint4* c4 = static_cast<uint4*>(a.best_cell);  // scratch, aligned to 256 bytes
    for (int i = first; i < a.n_cells / kVec; i += step) c4[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
    for (int i = a.n_cells / kVec * kVec + first; i < a.n_cells; i += step) cell[i] = kNone;
    for (int i = first; i < a.n_hits; i += step) hit[i] = kNone;
    return;
  }
  for (int i = first; i < n; i += step) {
    int row, nh;
    if (!candidate<T>(a, i, row, nh)) continue;
    const int32_t* C = a.cells + static_cast<int64_t>(row) * (kMaxHits - 1);
    for (int d = 0; d < nh - 1; ++d) cell[C[d]] = kNone;
    if (nh == 3) {
      const int32_t* H = a.hits + static_cast<int64_t>(row) * kMaxHits;
      for (int d = 0; d < 3; ++d) hit[H[d]] = kNone;
    }
  }
}

template <class T>
__global__ void __launch_bounds__(kBlock) k_amb_cell_min(AmbArgs a) {
  const int n = n_tracks(a);
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
    int row, nh;
    if (!candidate<T>(a, i, row, nh)) continue;
    const Key<T> k = key_of(static_cast<const T*>(a.chi2)[i]);
    const int32_t* C = a.cells + static_cast<int64_t>(row) * (kMaxHits - 1);
    for (int d = 0; d < nh - 1; ++d) atomicMin(static_cast<Key<T>*>(a.best_cell) + C[d], k);
  }
}

// The chi^2 rule; the triplets that pass it enter the minima of |d0| of
// their hits.
template <class T>
__global__ void __launch_bounds__(kBlock) k_amb_chi2_rule(AmbArgs a) {
  const int n = n_tracks(a);
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
    int row, nh;
    int f = 0;
    if (candidate<T>(a, i, row, nh)) {
      const Key<T> k = key_of(static_cast<const T*>(a.chi2)[i]);
      const Key<T>* best = static_cast<const Key<T>*>(a.best_cell);
      const int32_t* C = a.cells + static_cast<int64_t>(row) * (kMaxHits - 1);
      bool ok = true;
      for (int d = 0; d < nh - 1; ++d) ok = ok && best[C[d]] == k;
      if (ok && nh == 3) {
        const Key<T> t = key_of(static_cast<const T*>(a.params)[static_cast<int64_t>(i) * 5 + 3]);
        const int32_t* H = a.hits + static_cast<int64_t>(row) * kMaxHits;
        for (int d = 0; d < 3; ++d) atomicMin(static_cast<Key<T>*>(a.best_hit) + H[d], t);
        f = 2;
      } else {
        f = ok ? 1 : 0;
      }
    }
    a.flag[i] = f;
  }
}

// The |d0| rule among the triplets that passed the chi^2 rule.
template <class T>
__global__ void __launch_bounds__(kBlock) k_amb_tip_rule(AmbArgs a) {
  const int n = n_tracks(a);
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock) {
    if (a.flag[i] != 2) continue;
    const int row = a.kept ? a.kept[i] : i;
    const Key<T> t = key_of(static_cast<const T*>(a.params)[static_cast<int64_t>(i) * 5 + 3]);
    const Key<T>* best = static_cast<const Key<T>*>(a.best_hit);
    const int32_t* H = a.hits + static_cast<int64_t>(row) * kMaxHits;
    bool ok = true;
    for (int d = 0; d < 3; ++d) ok = ok && best[H[d]] == t;
    a.flag[i] = ok ? 1 : 0;
  }
}

__global__ void __launch_bounds__(kBlock) k_amb_list(AmbArgs a, int32_t* __restrict__ selected) {
  const int n = n_tracks(a);
  for (int i = blockIdx.x * kBlock + threadIdx.x; i < n; i += gridDim.x * kBlock)
    if (a.flag[i]) selected[a.pos[i]] = i;
}

}  // namespace

size_t ws_ambiguity(int n_hits, int cells_cap, int n_max) {
  Carver c(nullptr);
  c.take<uint64_t>(static_cast<size_t>(cells_cap));
  c.take<uint64_t>(static_cast<size_t>(n_hits));
  c.take<int32_t>(static_cast<size_t>(n_max));
  c.take<int32_t>(static_cast<size_t>(n_max) + 1);
  c.take<uint64_t>(scan_state_words(n_max));
  return c.off + 256;
}

pt_err launch_ambiguity(const pt_hits& h, const pt_cells& cells, const pt_ntuplets& T, int precision,
                        const pt_tracks& tracks, int32_t* selected, int32_t* n_selected, pt_workspace ws,
                        hipStream_t s) {
  const int n_max = std::min(T.cap, tracks.cap);
  Carver c(ws.ptr);
  AmbArgs a{};
  a.hits = T.hits;
  a.cells = T.cells;
  a.n = T.n;
  a.kept = T.kept;
  a.count = T.count;
  a.n_max = n_max;
  a.chi2 = tracks.chi2;
  a.params = tracks.params;
  a.n_hits = h.n_hits;
  a.n_cells = cells.cap;
  a.best_cell = c.take<uint64_t>(static_cast<size_t>(cells.cap));
  a.best_hit = c.take<uint64_t>(static_cast<size_t>(h.n_hits));
  a.flag = c.take<int32_t>(static_cast<size_t>(n_max));
  a.pos = c.take<int32_t>(static_cast<size_t>(n_max) + 1);
  a.state_words = static_cast<int32_t>(scan_state_words(n_max));
  a.state = c.take<uint64_t>(static_cast<size_t>(a.state_words));
  if (n_max == 0) return fill_i32(n_selected, 0, 1, s) == hipSuccess ? PT_OK : PT_ERR_DEVICE;
  const int g = grid_for(n_max, kBlock, 8192);
  const auto rules = [&](auto reset, auto cell_min, auto chi2_rule, auto tip_rule) {
    reset<<<g, kBlock, 0, s>>>(a);
    cell_min<<<g, kBlock, 0, s>>>(a);
    chi2_rule<<<g, kBlock, 0, s>>>(a);
    tip_rule<<<g, kBlock, 0, s>>>(a);
  };
  if (precision == PT_FIT_F64)
    rules(k_amb_reset<double>, k_amb_cell_min<double>, k_amb_chi2_rule<double>, k_amb_tip_rule<double>);
  else
    rules(k_amb_reset<float>, k_amb_cell_min<float>, k_amb_chi2_rule<float>, k_amb_tip_rule<float>);
  PT_LAUNCH_CHECK();
  PT_HIP_CHECK(exclusive_scan(a.flag, a.pos, n_max, a.count, ScanTotal{n_selected}, a.state, s));
  k_amb_list<<<g, kBlock, 0, s>>>(a, selected);
  PT_LAUNCH_CHECK();
  return PT_OK;
}

}  // namespace pt
