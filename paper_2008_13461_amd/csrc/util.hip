// Device-wide exclusive scan and fill kernels.
#include "pt_internal.h"

namespace pt {
namespace {

// n_dev, when given, holds the number of items actually present (<= n).
__device__ inline int64_t items(int64_t n, const int32_t* n_dev) {
  if (!n_dev) return n;
  const int64_t m = *n_dev;
  return m < 0 ? 0 : (m < n ? m : n);
}

// One tile per work-group, read and written as 16-byte vectors when VEC (src
// and dst 16-byte aligned).  One launch whatever the size: tile sums, a scan of
// them and a second pass over the data took three to five.
template <bool VEC>
__global__ void __launch_bounds__(kTileThreads) k_scan(const int32_t* __restrict__ src, int32_t* __restrict__ dst,
                                                       int64_t n, const int32_t* __restrict__ n_dev, uint64_t* state,
                                                       ScanTotal t) {
  __shared__ int32_t s_wave[kTileThreads / kWave + 1];
  n = items(n, n_dev);
  const int tile = blockIdx.x;
  const int64_t tiles = n > 0 ? (n + kTileItems - 1) / kTileItems : 1;
  if (tile >= tiles) return;
  const int64_t base = static_cast<int64_t>(tile) * kTileItems + threadIdx.x * kScanItems;
  int32_t v[kScanItems];
  load_items<VEC>(src, base, n, v);
  int32_t s = 0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) s = count_add(s, v[i]);
  int32_t end;
  int32_t run = tile_exclusive(s, tiles > 1 ? state : nullptr, tile, s_wave, &end, [&](int i) {
    int32_t x = 0;  // a tile before this one is full
    for (int q = __lane_id(); q < kTileItems; q += kWave) x = count_add(x, src[static_cast<int64_t>(i) * kTileItems + q]);
    return wave_count_sum(x);
  });
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    const int32_t x = v[i];
    v[i] = run;
    run = count_add(run, x);
  }
  store_items<VEC>(dst, base, n, v);
  if (tile == tiles - 1 && threadIdx.x == 0) {
    dst[n] = end;
    if (t.total) *t.total = end;
    if (end > t.cap) status_flag(t.status, t.flag);
  }
}

__global__ void __launch_bounds__(kTileThreads) k_tile_sums(const int32_t* __restrict__ data, int64_t n,
                                                            const int32_t* __restrict__ n_dev,
                                                            int32_t* __restrict__ sums) {
  __shared__ int32_t s_wave[kTileThreads / kWave + 1];
  n = items(n, n_dev);
  const int64_t first = static_cast<int64_t>(blockIdx.x) * kTileItems;
  int32_t s = 0;
  if (first + kTileItems <= n) {  // consecutive threads read consecutive items: the order does not matter
    int32_t v[kScanItems];
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) v[i] = data[first + i * kTileThreads + threadIdx.x];
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) s = count_add(s, v[i]);
  } else {
    for (int64_t at = first + threadIdx.x; at < n; at += kTileThreads) s = count_add(s, data[at]);
  }
  int32_t total;
  block_exclusive(s, s_wave, &total);
  if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

template <class T>
__global__ void k_fill(T* __restrict__ p, T v, int64_t n) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    p[i] = v;
}

}  // namespace

hipError_t exclusive_scan(const int32_t* src, int32_t* dst, int64_t n, const int32_t* n_dev, const ScanTotal& t,
                          uint64_t* state, hipStream_t s) {
  const unsigned tiles = static_cast<unsigned>(tiles_of(n, kTileItems));
  if (aligned16(src) && aligned16(dst))
    k_scan<true><<<tiles, kTileThreads, 0, s>>>(src, dst, n, n_dev, state, t);
  else
    k_scan<false><<<tiles, kTileThreads, 0, s>>>(src, dst, n, n_dev, state, t);
  return hipGetLastError();
}

hipError_t tile_sums(const int32_t* src, int64_t n, const int32_t* n_dev, int32_t* sums, hipStream_t s) {
  k_tile_sums<<<static_cast<unsigned>(tiles_of(n, kTileItems)), kTileThreads, 0, s>>>(src, n, n_dev, sums);
  return hipGetLastError();
}

hipError_t fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  k_fill<int32_t><<<grid_for(n, 256, 4096), 256, 0, s>>>(p, v, n);
  return hipGetLastError();
}

hipError_t fill_u8(uint8_t* p, uint8_t v, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  k_fill<uint8_t><<<grid_for(n, 256, 4096), 256, 0, s>>>(p, v, n);
  return hipGetLastError();
}

}  // namespace pt
