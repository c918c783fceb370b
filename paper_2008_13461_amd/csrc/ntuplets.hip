// n-tuplet search (paper section 3.2: root doublets, depth-first search over
// the cell graph, maximal paths only) and duplicate removal (section 3.3:
// among tracks sharing a hit doublet only those with the most hits stay).
//
// No output position comes from a shared counter (same-address atomics
// serialise on the device):
//  - roots: one kernel lists them in cell order, each work-group placing its
//    tile's after those of the tiles before (many tiles: count, scan, write);
//  - search: one thread per root walks the graph with an explicit stack of
//    at most max_hits - 1 cells, first counting the paths it emits, then,
//    after a scan over the roots that also lists those that emit any, writing
//    them at their final rows.  Rows therefore come out in root order and,
//    per root, in search order.
// Duplicate removal is order independent: every row raises the per-cell
// maximum of its length with atomicMax, then a row is kept when it attains
// the maximum on every one of its cells.
#include "pt_internal.h"

#include <algorithm>

namespace pt {
namespace {


struct TupIn {
  const int32_t* cell_inner;
  const int32_t* cell_outer;
  const uint8_t* cell_pair;
  const int32_t* cell_count;
  int32_t cells_cap;
  const int32_t* out_start;
  const int32_t* out_count;
  const int32_t* out_cell;
  const uint8_t* has_inner;
  int32_t links_cap;
  const int32_t* link_total;  // links found (the end of the last cell's run)
  int32_t* roots;
  int32_t* n_roots;
  int32_t cap;
  int32_t* hits;
  int32_t* cells;
  uint8_t* n;
  int32_t* count_raw;
  int32_t* kept;
  int32_t* count;
  int32_t* max_n;
  uint32_t* status;
};

// A cell with outer links (a root without any makes a 2-hit path) whose
// inner hit lies on a root layer, or on a layer whose cells are roots when
// no link ends on them; the inner hit's layer is the inner layer of the
// cell's pair.
__device__ inline bool is_root(const DevCfg& k, int out_count, int pair, bool free_) {
  const int L = k.pair_inner[pair];
  return out_count > 0 && (((k.root_always_mask >> L) & 1u) || (((k.root_if_free_mask >> L) & 1u) && free_));
}

// Root flags of the cells of a tile, in four runs: bit q of f[g] is the flag of
// cell base + 4 (g kTileThreads + thread) + q, every load issued up front.
constexpr int kRootRuns = kScanItems / 4;
static_assert(kRootRuns == 4, "four runs of groups of four");
template <bool VEC>
__device__ inline void group_flags(const DevCfg& k, const TupIn& a, int64_t base, int n, uint32_t (&f)[kRootRuns]) {
  if (VEC && base + kTileItems <= n) {
    int4 oc[kRootRuns];
    uint32_t pr[kRootRuns], hin[kRootRuns];
#pragma unroll
    for (int g = 0; g < kRootRuns; ++g) {
      const int64_t c0 = base + 4 * (g * kTileThreads + threadIdx.x);
      oc[g] = *reinterpret_cast<const int4*>(a.out_count + c0);
      pr[g] = *reinterpret_cast<const uint32_t*>(a.cell_pair + c0);
      hin[g] = *reinterpret_cast<const uint32_t*>(a.has_inner + c0);
    }
#pragma unroll
    for (int g = 0; g < kRootRuns; ++g) {
      const int o[4] = {oc[g].x, oc[g].y, oc[g].z, oc[g].w};
      f[g] = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        f[g] |= is_root(k, o[q], (pr[g] >> (8 * q)) & 0xFF, ((hin[g] >> (8 * q)) & 0xFF) == 0) ? 1u << q : 0u;
    }
    return;
  }
#pragma unroll
  for (int g = 0; g < kRootRuns; ++g) {
    f[g] = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t c = base + 4 * (g * kTileThreads + threadIdx.x) + q;
      if (c < n && is_root(k, a.out_count[c], a.cell_pair[c], !a.has_inner[c])) f[g] |= 1u << q;
    }
  }
}

// Lists the roots in cell order, one tile of kTileItems cells per work-group,
// in four runs of a group of four consecutive cells per thread.  VEC:
// out_count, cell_pair and has_inner 16- and 4-byte aligned; full tiles are
// then read four cells per load.
template <bool VEC>
__global__ void __launch_bounds__(kTileThreads) k_roots(DevCfg k, TupIn a, uint64_t* state) {
  __shared__ int32_t s_wave[2 * kTileThreads / kWave + 3];
  const int n = min(*a.cell_count, a.cells_cap);
  const int tiles = n > 0 ? (n + kTileItems - 1) / kTileItems : 1;
  const int tile = blockIdx.x;
  if (tile >= tiles) return;
  const int64_t base = static_cast<int64_t>(tile) * kTileItems;
  uint32_t f[kRootRuns];
  group_flags<VEC>(k, a, base, n, f);
  int c[kRootRuns], pos[kRootRuns], end;
#pragma unroll
  for (int g = 0; g < kRootRuns; ++g) c[g] = __popc(f[g]);
  tile_positions(c, tiles > 1 ? state : nullptr, tile, s_wave, pos, &end, [&](int i) {
    int x = 0;  // a tile before this one is full
    for (int q = __lane_id(); q < kTileItems; q += kWave) {
      const int64_t cell = static_cast<int64_t>(i) * kTileItems + q;
      x += is_root(k, a.out_count[cell], a.cell_pair[cell], !a.has_inner[cell]) ? 1 : 0;
    }
    return wave_sum(x);
  });
#pragma unroll
  for (int g = 0; g < kRootRuns; ++g) {
    int at = pos[g];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if ((f[g] >> q) & 1u) a.roots[at++] = static_cast<int>(base + 4 * (g * kTileThreads + threadIdx.x) + q);
  }
  if (tile == tiles - 1 && threadIdx.x == 0) *a.n_roots = end;
}

// The same in two steps around a scan, for many tiles: k_root_count counts the
// roots of each tile and stores their flags as a bit mask (bit b of word w is
// the flag of cell 64 w + b), and k_mask_write writes them from the mask,
// one wavefront per tile.
constexpr int kRootWords = kTileItems / kWave;  // mask words per tile
template <bool VEC>
__global__ void __launch_bounds__(kTileThreads) k_root_count(DevCfg k, TupIn a, int32_t* __restrict__ tile_roots,
                                                             uint64_t* __restrict__ bits) {
  __shared__ int32_t s_wave[kTileThreads / kWave + 1];
  __shared__ uint8_t s_f[kTileItems / 4];  // flags of each group of four cells
  const int n = min(*a.cell_count, a.cells_cap);
  const int64_t base = static_cast<int64_t>(blockIdx.x) * kTileItems;
  if (base >= n) {
    if (threadIdx.x == 0) tile_roots[blockIdx.x] = 0;
    return;
  }
  uint32_t f[kRootRuns];
  group_flags<VEC>(k, a, base, n, f);
  int cnt = 0;
#pragma unroll
  for (int g = 0; g < kRootRuns; ++g) {
    cnt += __popc(f[g]);
    s_f[g * kTileThreads + threadIdx.x] = static_cast<uint8_t>(f[g]);
  }
  int total;
  block_exclusive(cnt, s_wave, &total);  // its barriers also order the flags
  if (threadIdx.x < kRootWords) {        // 16 groups of four bits make a word
    const uint32_t* p = reinterpret_cast<const uint32_t*>(s_f) + 4 * threadIdx.x;
    uint64_t word = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t v = p[i];  // four groups, one byte each
      word |= static_cast<uint64_t>((v & 0xF) | (v >> 4 & 0xF0) | (v >> 8 & 0xF00) | (v >> 12 & 0xF000)) << (16 * i);
    }
    bits[blockIdx.x * static_cast<int64_t>(kRootWords) + threadIdx.x] = word;
  }
  if (threadIdx.x == 0) tile_roots[blockIdx.x] = total;
}

// Lane l holds word l of the tile: a root's position is the tile's offset,
// plus the set bits of the words before its own, plus its rank in its word.
__global__ void __launch_bounds__(kWave) k_mask_write(TupIn a, const uint64_t* __restrict__ bits,
                                                     const int32_t* __restrict__ tile_first) {
  static_assert(kRootWords == kWave, "one mask word per lane");
  const int n = min(*a.cell_count, a.cells_cap);
  const int64_t base = static_cast<int64_t>(blockIdx.x) * kTileItems;
  if (base >= n) return;
  const int lane = threadIdx.x;
  const uint64_t word = bits[blockIdx.x * static_cast<int64_t>(kRootWords) + lane];
  const int c = __popcll(word);
  const int first = tile_first[blockIdx.x] + wave_incl_scan(c) - c;  // this word's first root
  uint64_t nz = __ballot(word != 0);
  while (nz) {
    const int w = __builtin_ctzll(nz);
    nz &= nz - 1;
    const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(word), w);
    const uint32_t hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(word >> 32), w);
    const uint64_t m = (static_cast<uint64_t>(hi) << 32) | lo;
    const int at = __builtin_amdgcn_readlane(first, w);
    if ((m >> lane) & 1u) a.roots[at + lane_prefix(m)] = static_cast<int>(base + w * kWave + lane);
  }
}

// Lists the roots that emit a row below the capacity, with their first row,
// from the rows each root emits (paths[i], the count pass's output), one tile
// of kTileItems roots per work-group, kScanItems consecutive ones per thread;
// the list is in the order the work-groups come to it.  The last tile writes
// the total number of rows.
__global__ void __launch_bounds__(kTileThreads) k_first_rows(TupIn a, const int32_t* __restrict__ paths, uint64_t* state,
                                                             int2* __restrict__ prod, int32_t* __restrict__ n_prod) {
  __shared__ int32_t s_wave[kTileThreads / kWave + 1];
  __shared__ int32_t s_at;
  const int nr = min(*a.n_roots, a.cells_cap);
  const int tiles = nr > 0 ? (nr + kTileItems - 1) / kTileItems : 1;
  const int tile = blockIdx.x;
  if (tile >= tiles) return;
  const int64_t at = static_cast<int64_t>(tile) * kTileItems + static_cast<int64_t>(threadIdx.x) * kScanItems;
  int c[kScanItems];
  load_items<true>(paths, at, nr, c);  // scratch, 256-byte aligned
  int sum = 0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) sum = count_add(sum, c[i]);
  int end;
  const int first = tile_exclusive(sum, tiles > 1 ? state : nullptr, tile, s_wave, &end, [&](int i) {
    int x = 0;  // a tile before this one is full
    for (int q = __lane_id(); q < kTileItems; q += kWave)
      x = count_add(x, paths[static_cast<int64_t>(i) * kTileItems + q]);
    return wave_count_sum(x);
  });
  int run = first, cnt = 0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    cnt += c[i] > 0 && run < a.cap ? 1 : 0;  // at most a.cap roots in all: prod holds no more
    run = count_add(run, c[i]);
  }
  __syncthreads();  // s_wave is read
  int n_here;
  int w = block_exclusive(cnt, s_wave, &n_here);
  if (threadIdx.x == 0) s_at = n_here > 0 ? atomicAdd(n_prod, n_here) : 0;
  __syncthreads();
  w += s_at;
  run = first;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    if (c[i] > 0 && run < a.cap) prod[w++] = make_int2(static_cast<int>(at + i), run);
    run = count_add(run, c[i]);
  }
  if (tile == tiles - 1 && threadIdx.x == 0) {
    *a.count_raw = end;
    if (end > a.cap) status_flag(a.status, PT_FLAG_TUPLETS_OVERFLOW);
  }
}

// The run of cell c's outer links, [*first, *end): the links are placed in
// cell order, so the run ends where the next cell's starts (at the total
// after the last cell).  Both loads are issued together, so that a child's
// run comes one dependent load after its index instead of two.  Where the
// places have saturated, the count says whether the cell has links, which lie
// past the capacity (an end before the first: none to follow).
__device__ inline void link_run(const TupIn& a, int c, int n_cells, int total, int* first, int* end) {
  const int f = a.out_start[c];
  const int e = a.out_start[min(c + 1, n_cells - 1)];
  *first = f;
  *end = c + 1 < n_cells ? e : total;
  if (f == kMaxCount && a.out_count[c] > 0) *end = 0;
}

// Depth-first search from each root.  COUNT: paths[i] = rows root i emits
// (and the truncation count); otherwise the rows of the roots listed in prod
// are written from their first row on.
template <bool COUNT>
__global__ void k_dfs(DevCfg k, TupIn a, int32_t* __restrict__ paths, const int2* __restrict__ prod,
                      const int32_t* __restrict__ n_prod) {
  // the write pass takes only the roots that emit a row below the capacity
  // (most roots emit none: their paths are too short)
  const int nr = COUNT ? *a.n_roots : *n_prod;
  const int n_cells = min(*a.cell_count, a.cells_cap);
  const int links_found = *a.link_total;
  uint32_t truncated = 0;
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < nr; t += gridDim.x * blockDim.x) {
    int stack[kMaxHits];   // cells of the current path
    int next[kMaxHits];    // next outer link to follow at each depth (absolute link index) ...
    int end[kMaxHits];     // ... and the end of that cell's links
    const int2 from = COUNT ? make_int2(t, 0) : prod[t];  // the root's index, its first row
    const int root = a.roots[from.x];
    stack[0] = root;
    link_run(a, root, n_cells, links_found, &next[0], &end[0]);
    int depth = 0;
    int row = from.y;
    while (depth >= 0) {
      if (next[depth] >= end[depth]) {
        --depth;
        continue;
      }
      const int li = next[depth]++;
      if (li >= a.links_cap) continue;
      const int child = a.out_cell[li];
      const int nh = depth + 3;  // hits of the path root..child
      int cf, ce;
      link_run(a, child, n_cells, links_found, &cf, &ce);
      const int coc = ce - cf;
      if (coc == 0 || nh == k.max_hits) {
        if (COUNT && coc > 0) ++truncated;
        if (nh >= k.min_hits) {
          if (!COUNT && row < a.cap) {  // the cells of the path (its hits: k_row_hits)
            int32_t* C = a.cells + static_cast<int64_t>(row) * (kMaxHits - 1);
            for (int d = 0; d <= depth; ++d) {
              C[d] = stack[d];
              a.max_n[stack[d]] = 0;  // the only maxima read afterwards
            }
            C[depth + 1] = child;
            a.max_n[child] = 0;
            for (int d = depth + 2; d < kMaxHits - 1; ++d) C[d] = -1;
            a.n[row] = static_cast<uint8_t>(nh);
          }
          if (row < (COUNT ? kMaxCount : a.cap)) ++row;
        }
      } else {
        ++depth;
        stack[depth] = child;
        next[depth] = cf;
        end[depth] = ce;
      }
    }
    if (COUNT) paths[t] = row;
  }
  if (COUNT) {
    const uint32_t total = wave_status_add(a.status, PT_ST_TRUNCATED, truncated);
    if (total && __lane_id() == 0) status_flag(a.status, PT_FLAG_TRUNCATED);
  }
}

// The hits of every row from its cells (inner hit of the first cell, then
// the outer hit of each), one thread per row -- the search itself stores only
// the cells it holds in registers -- and the longest row through each cell.
__global__ void k_row_hits(TupIn a) {
  const int rows = min(*a.count_raw, a.cap);
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < rows; t += gridDim.x * blockDim.x) {
    const int nh = a.n[t];
    const int32_t* C = a.cells + static_cast<int64_t>(t) * (kMaxHits - 1);
    int c[kMaxHits - 1], h[kMaxHits];
#pragma unroll
    for (int d = 0; d < kMaxHits - 1; ++d) c[d] = C[d];
    h[0] = a.cell_inner[c[0]];
#pragma unroll
    for (int d = 0; d < kMaxHits - 1; ++d) h[d + 1] = d < nh - 1 ? a.cell_outer[c[d]] : -1;
    // Rows of one root are neighbours and share their first cells: a row leaves
    // a cell to the row before it in the wavefront when that is no shorter
    // (16 events with triplets: 562 -> 453 us, the atomics being most of it).
    const int before_n = __shfl_up(nh, 1, kWave);
    const bool leave = __lane_id() > 0 && before_n >= nh;
#pragma unroll
    for (int d = 0; d < kMaxHits - 1; ++d) {
      const int before = __shfl_up(c[d], 1, kWave);
      if (d < nh - 1 && !(leave && before == c[d])) atomicMax(a.max_n + c[d], nh);
    }
    int4* H = reinterpret_cast<int4*>(a.hits + static_cast<int64_t>(t) * kMaxHits);
    if (reinterpret_cast<uintptr_t>(a.hits) % 16 == 0) {
      H[0] = make_int4(h[0], h[1], h[2], h[3]);
      H[1] = make_int4(h[4], h[5], h[6], h[7]);
    } else {
#pragma unroll
      for (int d = 0; d < kMaxHits; ++d) a.hits[static_cast<int64_t>(t) * kMaxHits + d] = h[d];
    }
  }
}

// Lists the rows that attain the maximum on every one of their cells, in row
// order, one tile of kKeepTile rows per work-group, four per thread.  A
// thread's loads go out together, level by level (with 16 rows a thread, one
// after the other, an event's rows kept a handful of work-groups busy for 57
// us at pileup 200).  37 million rows, 36 000 tiles: 0.84 ms, where a count, a
// scan and a write took 1.36.
constexpr int kKeepTile = 4 * kTileThreads;
__global__ void __launch_bounds__(kTileThreads) k_keep(TupIn a, uint64_t* state) {
  __shared__ int32_t s_wave[2 * kTileThreads / kWave + 3];
  const int rows = min(*a.count_raw, a.cap);
  const int tiles = rows > 0 ? (rows + kKeepTile - 1) / kKeepTile : 1;
  const int tile = blockIdx.x;
  if (tile >= tiles) return;
  const int64_t base = static_cast<int64_t>(tile) * kKeepTile + threadIdx.x;
  int nh[4], keep[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) nh[i] = base + i * kTileThreads < rows ? a.n[base + i * kTileThreads] : 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int32_t* C = a.cells + (base + i * kTileThreads) * (kMaxHits - 1);
    int c[kMaxHits - 1], best[kMaxHits - 1];
#pragma unroll
    for (int d = 0; d < kMaxHits - 1; ++d) c[d] = d < nh[i] - 1 ? C[d] : -1;
#pragma unroll
    for (int d = 0; d < kMaxHits - 1; ++d) best[d] = c[d] >= 0 ? a.max_n[c[d]] : nh[i];
    bool ok = nh[i] > 0;
#pragma unroll
    for (int d = 0; d < kMaxHits - 1; ++d) ok = ok && best[d] == nh[i];
    keep[i] = ok ? 1 : 0;
  }
  int pos[4], end;
  tile_positions(keep, tiles > 1 ? state : nullptr, tile, s_wave, pos, &end, [&](int i) {
    int x = 0;  // a tile before this one is full
    for (int q = __lane_id(); q < kKeepTile; q += kWave) {
      const int64_t t = static_cast<int64_t>(i) * kKeepTile + q;
      bool ok = true;
      for (int d = 0; d < a.n[t] - 1; ++d) ok = ok && a.max_n[a.cells[t * (kMaxHits - 1) + d]] == a.n[t];
      x += ok ? 1 : 0;
    }
    return wave_sum(x);
  });
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (keep[i]) a.kept[pos[i]] = static_cast<int>(base + i * kTileThreads);
  if (tile == tiles - 1 && threadIdx.x == 0) *a.count = end;
}

}  // namespace

// Scratch words cleared at the start of a call: the states of the three
// listings and the number of roots that emit rows.  With many cells the roots'
// are those of the scan over the tiles, a part of them.
static size_t state_words(int cells_cap, int tuplets_cap) {
  return 2 * scan_state_words(cells_cap) + tiles_of(tuplets_cap, kKeepTile) + 1;
}
static size_t mask_tiles(int cells_cap) { return cells_cap > kLargeItems ? tiles_of(cells_cap, kTileItems) : 0; }

size_t ws_ntuplets(int cells_cap, int tuplets_cap) {
  Carver c(nullptr);
  c.take<uint64_t>(state_words(cells_cap, tuplets_cap));
  c.take<int32_t>(1);              // number of roots
  c.take<int32_t>(cells_cap);      // roots
  c.take<int2>(tuplets_cap);       // roots that emit rows, with their first row (each has one below the capacity)
  c.take<int32_t>(cells_cap);      // paths per root
  c.take<int32_t>(cells_cap);      // max_n
  c.take<uint64_t>(mask_tiles(cells_cap) * kRootWords);  // root flags, one bit per cell
  c.take<int32_t>(mask_tiles(cells_cap));                // roots per tile
  c.take<int32_t>(mask_tiles(cells_cap) + 1);            // first root of each tile
  return c.off + 256;
}

pt_err launch_ntuplets(const pt_hits& h, const DevCfg& k, const pt_cells& in_cells, const pt_links& in_links,
                       pt_ntuplets& out, uint32_t* status, pt_workspace ws, hipStream_t s) {
  (void)h;
  pt_cells cells = in_cells;
  pt_links L = in_links;
  pt_ntuplets T = out;
  cells.cap = capacity(in_cells.cap);
  L.cap = capacity(in_links.cap);
  T.cap = capacity(out.cap);
  Carver c(ws.ptr);
  const size_t words = state_words(cells.cap, T.cap);
  uint64_t* state = c.take<uint64_t>(words);
  int32_t* n_roots = c.take<int32_t>(1);
  int32_t* roots = c.take<int32_t>(cells.cap);
  int2* prod = c.take<int2>(T.cap);
  int32_t* paths = c.take<int32_t>(cells.cap);
  int32_t* max_n = c.take<int32_t>(cells.cap);
  const size_t n_mask = mask_tiles(cells.cap);
  uint64_t* bits = c.take<uint64_t>(n_mask * kRootWords);
  int32_t* tile_roots = c.take<int32_t>(n_mask);
  int32_t* tile_first = c.take<int32_t>(n_mask + 1);
  uint64_t* root_state = state;
  uint64_t* row_state = root_state + scan_state_words(cells.cap);
  uint64_t* keep_state = row_state + scan_state_words(cells.cap);
  int32_t* n_prod = reinterpret_cast<int32_t*>(keep_state + tiles_of(T.cap, kKeepTile));
  TupIn a{cells.inner, cells.outer, cells.pair, cells.count, cells.cap, L.out_start, L.out_count, L.out_cell,
          L.has_inner, L.cap, L.count, roots, n_roots, T.cap, T.hits, T.cells, T.n, T.count_raw, T.kept, T.count,
          max_n, status};
  void* tok = timing_begin(s);
  PT_HIP_CHECK(fill_i32(reinterpret_cast<int32_t*>(state), 0, static_cast<int64_t>(2 * words), s));
  const unsigned tiles = static_cast<unsigned>(tiles_of(cells.cap, kTileItems));
  const bool vec = aligned16(L.out_count) && reinterpret_cast<uintptr_t>(cells.pair) % 4 == 0 &&
                   reinterpret_cast<uintptr_t>(L.has_inner) % 4 == 0;
  if (n_mask) {
    if (vec)
      k_root_count<true><<<tiles, kTileThreads, 0, s>>>(k, a, tile_roots, bits);
    else
      k_root_count<false><<<tiles, kTileThreads, 0, s>>>(k, a, tile_roots, bits);
    PT_LAUNCH_CHECK();
    PT_HIP_CHECK(exclusive_scan(tile_roots, tile_first, static_cast<int64_t>(n_mask), nullptr, ScanTotal{n_roots},
                                root_state, s));
  }
  timing_end(tok, "root_count", s);
  tok = timing_begin(s);
  if (n_mask)
    k_mask_write<<<tiles, kWave, 0, s>>>(a, bits, tile_first);
  else if (vec)
    k_roots<true><<<tiles, kTileThreads, 0, s>>>(k, a, root_state);
  else
    k_roots<false><<<tiles, kTileThreads, 0, s>>>(k, a, root_state);
  timing_end(tok, "root_write", s);
  PT_LAUNCH_CHECK();
  tok = timing_begin(s);
  k_dfs<true><<<grid_for(cells.cap, 256, 65536), 256, 0, s>>>(k, a, paths, nullptr, nullptr);
  timing_end(tok, "dfs_count", s);
  PT_LAUNCH_CHECK();
  tok = timing_begin(s);
  k_first_rows<<<static_cast<unsigned>(tiles_of(cells.cap, kTileItems)), kTileThreads, 0, s>>>(a, paths, row_state, prod,
                                                                                             n_prod);
  PT_LAUNCH_CHECK();
  k_dfs<false><<<grid_for(cells.cap, 128, 16384), 128, 0, s>>>(k, a, nullptr, prod, n_prod);
  timing_end(tok, "dfs_write", s);
  PT_LAUNCH_CHECK();
  tok = timing_begin(s);
  k_row_hits<<<grid_for(T.cap, 256, 8192), 256, 0, s>>>(a);
  PT_LAUNCH_CHECK();
  k_keep<<<static_cast<unsigned>(tiles_of(T.cap, kKeepTile)), kTileThreads, 0, s>>>(a, keep_state);
  PT_LAUNCH_CHECK();
  timing_end(tok, "dedup", s);
  return PT_OK;
}

}  // namespace pt
