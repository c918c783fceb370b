// Fishbone (paper section 3.3): among the doublets that share their outer
// hit, the longer of two aligned ones is dropped, so that the overlapping
// modules of a layer give one n-tuplet per particle instead of several.
//
// Runs inside pt_build_doublets when the Fishbone is on; the doublet step then
// writes its cells to the workspace:
//   1. the stored cells are indexed by outer hit with the index of the link
//      step (blocks of consecutive cells grouped by outer hit in LDS, one
//      segment per block and hit; no per-cell atomic);
//   2. a team of threads per outer hit gathers the hit's cells into LDS,
//      counting-sorted by a polar-direction key of the vector to the outer hit
//      into buckets at least as wide as the cut angle, and tests each cell
//      only against the cells of its own and the neighbouring buckets (and of
//      those around its negated key: nearly opposite vectors); a dot product
//      in single precision filters the pairs, the exact test, in double,
//      decides and clears the cell's keep flag.  Hits with more cells than a
//      team stages are listed for the next larger one;
//   3. the kept cells are written to the output in their order, in one pass
//      over the flags (the sum of the tiles before comes with it), and each
//      inner hit's range of cells is moved with them.
// The test is the one of pixeltrack.h, in double, as parenthesised, without
// contraction, from the hits' coordinates promoted to double.
#include <algorithm>
#include <cmath>
#include <mutex>

#include "pt_internal.h"

#pragma clang fp contract(off)

namespace pt {
namespace {

constexpr int kBlock = 256;
constexpr int kTiers = 3;  // kernels that stage an outer hit's cells in LDS, by their number:
constexpr int kTierCap[kTiers] = {256, 512, 1024};           // at most so many ...
constexpr int kTierTeam[kTiers] = {kWave, 2 * kWave, kBlock};  // ... with so many threads
constexpr int kNB = 256;       // most key buckets
constexpr int32_t kHitMask = 0x7fffffff;

template <class T>
struct FbArgs {
  const T* x;
  const T* y;
  const T* z;
  int32_t n_hits;
  double theta2;
  int32_t nb;             // key buckets: each at least the cut angle wide
  float kwin;             // key window: asin(theta) with a margin, 2 when theta >= 1
  float cos2_min;         // squared cosine, in single precision, below which two vectors are not aligned
  const int32_t* found;   // cells found
  int32_t cap;
  const int32_t* inner;   // the cells as found
  const int32_t* outer;
  const uint8_t* pair;
  int32_t* inner_first;
  int32_t* inner_count;
  OuterIndex idx;
  // workspace
  uint8_t* keep;          // [cap, a multiple of 16] flags
  int32_t* before;        // [cap / 16] kept cells before each group of 16
  int32_t* list[kTiers];  // [n_hits] outer hits with more cells than tier i stages
  int32_t* n_list;        // [kTiers] how many
  int32_t* out_inner;     // the output cells
  int32_t* out_outer;
  uint8_t* out_pair;
  int32_t* out_count;
  uint64_t* state;        // of the scan of the flags
  int32_t state_words;
};

// Cells the Fishbone works on: every stored cell, or none when the cells
// overflowed their capacity (the products are truncated anyway).
template <class T>
__device__ inline int stored(const FbArgs<T>& a) {
  const int c = *a.found;
  return c <= a.cap ? c : 0;
}

// Squared lengths, in single precision, of which a unit vector and a key are
// formed; below the keys, the mark of a hit with a vector out of the range.
constexpr float kMinLen2 = 1e-30f, kMaxLen2 = 1e30f, kEvery = -2.f;

// Polar-direction key of a vector: uz / (|u_T| + |uz|), in [-1, 1].  As a
// function of the angle to the z axis its slope is at most 1, and two
// vectors at an angle a differ in that angle by at most a, so their keys
// differ by at most a (for nearly opposite vectors, at an angle pi - a, the
// sum of their keys is at most a in magnitude).  NaN, which is never too far
// from another key, for a vector out of the range.
__device__ inline float polar_key(double ux, double uy, double uz) {
  const float l2 = float((ux * ux + uy * uy) + uz * uz);
  if (!(l2 > kMinLen2 && l2 < kMaxLen2)) return __builtin_nanf("");
  const float t = sqrtf(float(ux * ux + uy * uy));
  return float(uz) / (t + fabsf(float(uz)));
}

// Bucket of a key in [-1, 1] among nb buckets of width 2 / nb.
__device__ inline int bucket(float k, int nb) {
  const int b = static_cast<int>((k + 1.f) * (0.5f * static_cast<float>(nb)));
  return b < 0 ? 0 : (b >= nb ? nb - 1 : b);
}

// The exact test: the cell with vector u (length^2 U2) is dropped by a
// shorter cell of vector v when they are aligned.
__device__ inline bool kills(double ux, double uy, double uz, double U2, double vx, double vy, double vz,
                             double V2, double theta2) {
  if (!(V2 < U2)) return false;
  const double wx = uy * vz - uz * vy, wy = uz * vx - ux * vz, wz = ux * vy - uy * vx;
  const double W2 = (wx * wx + wy * wy) + wz * wz;
  return W2 <= theta2 * (U2 * V2);
}

template <class T>
__device__ inline void vec_to(const FbArgs<T>& a, double Xh, double Yh, double Zh, int i, double& ux, double& uy,
                           double& uz, double& U2) {
  ux = Xh - double(a.x[i]);
  uy = Yh - double(a.y[i]);
  uz = Zh - double(a.z[i]);
  U2 = (ux * ux + uy * uy) + uz * uz;
}

template <class T>
__global__ void k_fb_flags(FbArgs<T> a) {
  const int n = min(*a.found, a.cap);
  const int first = blockIdx.x * blockDim.x + threadIdx.x, step = gridDim.x * blockDim.x;
  for (int64_t c = first; 16 * c < n; c += step)
    reinterpret_cast<int4*>(a.keep)[c] = make_int4(0x01010101, 0x01010101, 0x01010101, 0x01010101);
  for (int i = first; i < a.state_words; i += step) a.state[i] = 0;
  if (first < kTiers) a.n_list[first] = 0;
}

// Barrier and reductions over the TEAM threads (a wavefront, or the whole
// block) that work on one outer hit.
template <int TEAM>
__device__ __forceinline__ void team_sync() {
  if constexpr (TEAM == kWave) wave_sync(); else __syncthreads();
}

// Inclusive prefix sum of v over the team, the total to *total; s_w holds
// one word per wavefront of the team.
template <int TEAM>
__device__ inline int team_scan(int v, int32_t* s_w, int* total) {
  const int incl = wave_incl_scan(v);
  if constexpr (TEAM == kWave) {
    *total = __builtin_amdgcn_readlane(incl, kWave - 1);
    return incl;
  } else {
    const int wave = static_cast<int>(threadIdx.x % TEAM) / kWave;
    __syncthreads();  // the words of the previous scan are read
    if (__lane_id() == kWave - 1) s_w[wave] = incl;
    __syncthreads();
    int before = 0, sum = 0;
#pragma unroll
    for (int w = 0; w < TEAM / kWave; ++w) {
      if (w < wave) before += s_w[w];
      sum += s_w[w];
    }
    *total = sum;
    return before + incl;
  }
}

// Minimum of v over the team (s_w as in team_scan).
template <int TEAM>
__device__ inline float team_min(float v, float* s_w) {
  v = wave_min(v);
  if constexpr (TEAM > kWave) {
    const int wave = static_cast<int>(threadIdx.x % TEAM) / kWave;
    __syncthreads();
    if (__lane_id() == 0) s_w[wave] = v;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < TEAM / kWave; ++w) v = fminf(v, s_w[w]);
  }
  return v;
}

// The cells of one outer hit by one team of threads, a work-group: a
// wavefront for every hit with at most kTierCap[0] cells (tier 0; hits differ
// in their cells by orders of magnitude, and a work-group of four wavefronts,
// a hit each, held its slots until the slowest was done: 1.83 against 2.25
// ms), and two or four for the hits with more, which the tier before lists (a
// persistent grid; two against four for 257..512 cells: 1.29 against 1.48 ms).
//
// The cells are staged in LDS sorted by key bucket -- the unit vector to the
// outer hit and its squared length in one 16-byte vector, the inner hit's
// coordinates beside it -- so that a cell's candidates are contiguous and
// neighbouring lanes, which take neighbouring cells of the sorted list, scan
// nearly the same ones, four a step.  A candidate costs one LDS read and a
// dot product in single precision: 1 - (n_i . n_j)^2 is the squared sine to
// 2e-6, so that only pairs within the cut angle and not longer go on to the
// exact test (in double, from the coordinates), which then nearly always
// decides and is run by all lanes that found such a pair together.  With a
// coarse azimuth filter in its place, some lane of the wavefront ran the
// exact test in nearly every step (16 PU200 overlap events, the two kernels:
// 9.4 ms against 3.0).  Meeting each pair once and queueing the
// aligned ones for full wavefronts of exact tests took 3.5 ms: a cell has 3.2
// aligned partners, and the first already decides.
template <class T, int TIER>
__global__ void __launch_bounds__(kTierTeam[TIER]) k_fb_kill(FbArgs<T> a) {
  constexpr int CAP = kTierCap[TIER], TEAM = kTierTeam[TIER];
  constexpr bool LISTED = TIER > 0;
  constexpr int kRounds = CAP / TEAM;
  constexpr int kStep = 4;  // candidates per step of a scan
  static_assert(CAP % TEAM == 0, "whole rounds");
  __shared__ float4 s_vec[CAP + kStep];  // by bucket: unit vector, squared length (NaN: in every test)
  __shared__ T s_x[CAP];                 // by bucket: the inner hit
  __shared__ T s_y[CAP];
  __shared__ T s_z[CAP];
  __shared__ int32_t s_cell[CAP];        // by bucket: the cell
  __shared__ uint8_t s_bk[CAP];          // by bucket: the bucket
  __shared__ int32_t s_bin[kNB + 1];     // cells per bucket, then first position
  __shared__ int32_t s_sum[TEAM / kWave];
  __shared__ float s_min[TEAM / kWave];
  int32_t* s_base = reinterpret_cast<int32_t*>(s_vec);  // while the cells are gathered: per segment
  int32_t* s_mark = s_cell;                             // ... and per cell its segment's index
  const int t = static_cast<int>(threadIdx.x);
  const int n_items = LISTED ? a.n_list[max(TIER - 1, 0)] : a.n_hits;
  if (stored(a) == 0) return;
  const int nb = a.nb;
  for (int item = blockIdx.x; item < n_items; item += LISTED ? gridDim.x : n_items) {
    const int h = LISTED ? a.list[max(TIER - 1, 0)][item] : item;
    const int sb = a.idx.seg_first[h], se = a.idx.seg_first[h + 1];
    const double Xh = double(a.x[h]), Yh = double(a.y[h]), Zh = double(a.z[h]);
    // the hit's cells, from the sizes of its segments
    const int2 g0 = sb + t < se ? a.idx.seg[sb + t] : make_int2(0, 0);
    int at;
    const int i0 = team_scan<TEAM>(g0.y, s_sum, &at);
    int m = at;
    for (int s0 = sb + TEAM; s0 < se; s0 += TEAM) {
      int more;
      team_scan<TEAM>(s0 + t < se ? a.idx.seg[s0 + t].y : 0, s_sum, &more);
      m += more;
    }
    if (m < 2) continue;
    if (m > CAP) {  // more cells than this kernel stages: listed for the next
      if (t == 0) a.list[TIER][atomicAdd(a.n_list + TIER, 1)] = h;
      continue;
    }
    team_sync<TEAM>();  // the previous hit's LDS is no longer read
    // the index entry of each cell: a segment marks its first cell and its
    // first in every 64, and a maximum over the 64 before finds a cell's mark
    for (int f = t; f < m; f += TEAM) s_mark[f] = -1;
    for (int b = t; b <= nb; b += TEAM) s_bin[b] = 0;
    team_sync<TEAM>();
    auto mark = [&](int s, int2 g, int first) {
      if (g.y > 0) {
        s_base[s] = g.x - first;
        for (int f = first; f < first + g.y; f = (f / kWave + 1) * kWave) s_mark[f] = s;
      }
    };
    mark(t, g0, i0 - g0.y);
    for (int s0 = TEAM; s0 < se - sb; s0 += TEAM) {
      const int2 g = sb + s0 + t < se ? a.idx.seg[sb + s0 + t] : make_int2(0, 0);
      int more;
      const int incl = team_scan<TEAM>(g.y, s_sum, &more);
      mark(s0 + t, g, at + incl - g.y);
      at += more;
    }
    team_sync<TEAM>();
    int cell[kRounds], ih[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      const int f = r * TEAM + t;
      cell[r] = -1;
      if (r * TEAM < m) {  // uniform
        const int s = wave_max_scan(f < m ? s_mark[f] : -1);
        if (f < m) {
          const int2 en = a.idx.ent[s_base[s] + f];
          cell[r] = en.x;
          ih[r] = en.y & kHitMask;
        }
      }
    }
    T px[kRounds], py[kRounds], pz[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      if (cell[r] >= 0) {
        px[r] = a.x[ih[r]];
        py[r] = a.y[ih[r]];
        pz[r] = a.z[ih[r]];
      }
    }
    // the cells' vectors, in registers until their places are known
    const float rh = sqrtf(float(Xh) * float(Xh) + float(Yh) * float(Yh));
    const float hx = rh > 0.f ? float(Xh) / rh : 0.f, hy = rh > 0.f ? float(Yh) / rh : 0.f;
    const float zs = Zh < 0.0 ? -1.f : 1.f;
    float rmin = 2.f, zmin = 2.f;  // smallest radial and z-side keys of the thread's cells
    float4 vec[kRounds];
    int place[kRounds];  // bucket | rank in it << 8
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      if (cell[r] < 0) continue;
      const double dx = Xh - double(px[r]), dy = Yh - double(py[r]), dz = Zh - double(pz[r]);
      const float ux = float(dx), uy = float(dy), uz = float(dz);
      const float t2 = ux * ux + uy * uy;
      // polar key: uz / (|u_T| + |uz|)
      const float l = sqrtf(t2) + fabsf(uz);
      const float kz = l > 0.f ? uz / l : 0.f;
      const int b = bucket(kz, nb);
      place[r] = b | (atomicAdd(&s_bin[b], 1) << 8);
      // key of the vector about the outer hit's transverse direction
      const float ur = ux * hx + uy * hy;
      const float ox = ux - ur * hx, oy = uy - ur * hy;
      const float lr = sqrtf(ox * ox + oy * oy + uz * uz) + fabsf(ur);
      rmin = fminf(rmin, lr > 0.f ? ur / lr : 0.f);
      zmin = fminf(zmin, kz * zs);
      // the length is rounded once, so that it never orders two the wrong
      // way; one whose square is out of range (a doublet of no length is
      // aligned with every other) takes part in every test of the hit
      float l2 = float((dx * dx + dy * dy) + dz * dz);
      if (!(l2 > kMinLen2 && l2 < kMaxLen2)) {
        l2 = __builtin_nanf("");
        rmin = kEvery;
      }
      const float inv = __builtin_amdgcn_rsqf(l2);
      vec[r] = make_float4(ux * inv, uy * inv, uz * inv, l2);
    }
    // nearly opposite partners are possible only when neither family of keys
    // stays above the cut angle for every cell of the hit (two nearly opposite
    // vectors cannot both point away from the beam line, or both along the
    // outer hit's side of z, by more than the cut angle)
    rmin = team_min<TEAM>(rmin, s_min);
    const bool every = rmin == kEvery;  // no buckets: each cell against all
    const bool mirror = !every && rmin <= a.kwin && team_min<TEAM>(zmin, s_min) <= a.kwin;
    team_sync<TEAM>();
    if (t < kWave) {  // first positions: a scan over the buckets
      int carry = 0;
      for (int b0 = 0; b0 < nb; b0 += kWave) {
        const int b = b0 + t;
        const int c = b < nb ? s_bin[b] : 0;
        const int incl = wave_incl_scan(c);
        if (b < nb) s_bin[b] = carry + incl - c;
        carry += __builtin_amdgcn_readlane(incl, kWave - 1);
      }
      if (t == 0) s_bin[nb] = carry;
    }
    team_sync<TEAM>();
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
      if (cell[r] < 0) continue;
      const int b = place[r] & 0xFF;
      const int p = s_bin[b] + (place[r] >> 8);
      s_vec[p] = vec[r];
      s_x[p] = px[r];
      s_y[p] = py[r];
      s_z[p] = pz[r];
      s_cell[p] = cell[r];
      s_bk[p] = static_cast<uint8_t>(b);
    }
    team_sync<TEAM>();
    // each cell against the cells of its bucket and the two next to it, and of
    // the buckets around its negated key (nearly opposite vectors)
    for (int p = t; p < m; p += TEAM) {
      const float4 u = s_vec[p];
      const int b = s_bk[p];
      bool killed = false;
      for (int pass = 0; pass < (mirror ? 2 : 1) && !killed; ++pass) {
        const int c = pass == 0 ? b : nb - 1 - b;
        int q = every ? 0 : s_bin[max(c - 1, 0)];
        const int q1 = every ? m : s_bin[min(c + 2, nb)];
        while (q < q1) {
          // the next candidates within the cut angle and not longer
          uint32_t found = 0;
          for (; q < q1; q += kStep) {
#pragma unroll
            for (int k = 0; k < kStep; ++k) {
              const float4 v = s_vec[q + k];
              const float d = __builtin_fmaf(u.z, v.z, __builtin_fmaf(u.y, v.y, u.x * v.x));
              if (!(d * d < a.cos2_min) && !(v.w > u.w)) found |= 1u << k;
            }
            found &= (2u << min(q1 - q - 1, kStep - 1)) - 1u;                         // not past the range
            found &= ~(static_cast<uint32_t>(p - q) < kStep ? 1u << (p - q) : 0u);  // nor itself
            if (found) break;
          }
          const double ux = Xh - double(s_x[p]), uy = Yh - double(s_y[p]), uz = Zh - double(s_z[p]);
          const double U2 = (ux * ux + uy * uy) + uz * uz;
          while (found) {
            const int j = q + __builtin_ctz(found);
            found &= found - 1;
            const double vx = Xh - double(s_x[j]), vy = Yh - double(s_y[j]), vz = Zh - double(s_z[j]);
            killed = kills(ux, uy, uz, U2, vx, vy, vz, (vx * vx + vy * vy) + vz * vz, a.theta2);
            if (killed) found = 0;
          }
          q = killed ? q1 : q + kStep;
        }
      }
      if (killed) a.keep[s_cell[p]] = 0;
    }
  }
}

// The outer hits with more cells than the last tier stages, one work-group each (a
// persistent grid over the list): the hit's cells are staged in LDS (up to
// kBigCap; beyond, from global memory) and each thread tests its cells
// against all the others of the hit whose key is within the cut angle of
// its own or of its negative.
constexpr int kBigBlock = 1024;
constexpr int kBigCap = 3072;
constexpr int kBigSegs = 1024;

template <class T>
__global__ void __launch_bounds__(kBigBlock) k_fb_kill_big(FbArgs<T> a) {
  __shared__ T s_x[kBigCap], s_y[kBigCap], s_z[kBigCap];
  __shared__ float s_k[kBigCap];
  __shared__ int32_t s_cell[kBigCap];
  __shared__ int32_t s_start[kBigSegs + 1];
  const int nbig = a.n_list[kTiers - 1];
  const float win = a.kwin;
  for (int b = blockIdx.x; b < nbig; b += gridDim.x) {
    const int h = a.list[kTiers - 1][b];
    const int sb = a.idx.seg_first[h], ns = a.idx.seg_first[h + 1] - sb;
    const double Xh = double(a.x[h]), Yh = double(a.y[h]), Zh = double(a.z[h]);
    __syncthreads();  // the previous hit's LDS is no longer read
    if (threadIdx.x == 0) {
      int run = 0;
      for (int q = 0; q < ns && q < kBigSegs; ++q) {
        s_start[q] = run;
        run += a.idx.seg[sb + q].y;
      }
      s_start[min(ns, kBigSegs)] = run;
    }
    __syncthreads();
    const int m = s_start[min(ns, kBigSegs)];
    if (ns <= kBigSegs && m <= kBigCap) {
      for (int f = threadIdx.x; f < m; f += kBigBlock) {
        int l = 0, r = ns - 1;  // the last segment starting at or before f
        while (l < r) {
          const int mid = (l + r + 1) >> 1;
          if (s_start[mid] <= f) l = mid; else r = mid - 1;
        }
        const int2 en = a.idx.ent[a.idx.seg[sb + l].x + (f - s_start[l])];
        const int ih = en.y & kHitMask;
        const T hx = a.x[ih], hy = a.y[ih], hz = a.z[ih];
        s_cell[f] = en.x;
        s_x[f] = hx;
        s_y[f] = hy;
        s_z[f] = hz;
        s_k[f] = polar_key(Xh - double(hx), Yh - double(hy), Zh - double(hz));
      }
      __syncthreads();
      for (int i = threadIdx.x; i < m; i += kBigBlock) {
        const double ux = Xh - double(s_x[i]), uy = Yh - double(s_y[i]), uz = Zh - double(s_z[i]);
        const double U2 = (ux * ux + uy * uy) + uz * uz;
        const float ki = s_k[i];
        bool killed = false;
        for (int j = 0; j < m && !killed; ++j) {
          const float kj = s_k[j];
          if (j == i || (fabsf(kj - ki) > win && fabsf(kj + ki) > win)) continue;
          const double vx = Xh - double(s_x[j]), vy = Yh - double(s_y[j]), vz = Zh - double(s_z[j]);
          const double V2 = (vx * vx + vy * vy) + vz * vz;
          killed = kills(ux, uy, uz, U2, vx, vy, vz, V2, a.theta2);
        }
        if (killed) a.keep[s_cell[i]] = 0;
      }
    } else {
      // beyond the LDS: every pair from global memory, threads over the
      // hit's cells segment by segment
      for (int s = 0; s < ns; ++s) {
        const int2 gi = a.idx.seg[sb + s];
        for (int e = threadIdx.x; e < gi.y; e += kBigBlock) {
          const int2 en = a.idx.ent[gi.x + e];
          double ux, uy, uz, U2;
          vec_to(a, Xh, Yh, Zh, en.y & kHitMask, ux, uy, uz, U2);
          bool killed = false;
          for (int t = 0; t < ns && !killed; ++t) {
            const int2 gj = a.idx.seg[sb + t];
            for (int f = 0; f < gj.y && !killed; ++f) {
              const int2 ej = a.idx.ent[gj.x + f];
              if (ej.x == en.x) continue;
              double vx, vy, vz, V2;
              vec_to(a, Xh, Yh, Zh, ej.y & kHitMask, vx, vy, vz, V2);
              killed = kills(ux, uy, uz, U2, vx, vy, vz, V2, a.theta2);
            }
          }
          if (killed) a.keep[en.x] = 0;
        }
      }
    }
  }
}

// The 16 flags of cells 16 g .. 16 g + 15 below n as a bit mask.
template <class T>
__device__ inline uint32_t flags16(const FbArgs<T>& a, int64_t g, int n) {
  const int left = n - static_cast<int>(16 * g);
  if (left <= 0) return 0;
  const int4 q = reinterpret_cast<const int4*>(a.keep)[g];
  const uint32_t w[4] = {static_cast<uint32_t>(q.x), static_cast<uint32_t>(q.y), static_cast<uint32_t>(q.z),
                         static_cast<uint32_t>(q.w)};
  uint32_t m = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) m |= ((w[k] * 0x10204080u) >> 28) << (4 * k);  // byte b's bit 0 to bit b
  return left < 16 ? m & ((1u << left) - 1u) : m;
}

// Writes the kept cells to the output in their order, one tile of kTileItems
// cells per work-group, and the kept cells before each 16 for the ranges.
// One thread's 16 flags give the positions of 16 consecutive cells; the cells
// themselves go one per thread and round, through LDS, so that loads and
// stores stay coalesced.
template <class T>
__global__ void __launch_bounds__(kTileThreads) k_fb_compact(FbArgs<T> a) {
  static_assert(kScanItems == 16, "a thread's flags are one 16-byte vector");
  __shared__ int32_t s_wave[kTileThreads / kWave + 1];
  __shared__ int32_t s_at[kTileThreads];    // per 16 cells: kept ones before
  __shared__ uint32_t s_m[kTileThreads];    // ... and their flags
  const int found = *a.found;
  const int n = min(found, a.cap);
  const int tiles = n > 0 ? (n + kTileItems - 1) / kTileItems : 1;
  const int tile = blockIdx.x;
  if (tile >= tiles) return;
  const int t = threadIdx.x;
  const int64_t g0 = static_cast<int64_t>(tile) * kTileThreads;
  const uint32_t m = flags16(a, g0 + t, n);
  int end;
  const int at = tile_exclusive(__popc(m), tiles > 1 ? a.state : nullptr, tile, s_wave, &end, [&](int i) {
    int x = 0;  // a tile before this one is full
    for (int q = __lane_id(); q < kTileThreads; q += kWave)
      x += __popc(flags16(a, static_cast<int64_t>(i) * kTileThreads + q, n));
    return wave_sum(x);
  });
  s_at[t] = at;
  s_m[t] = m;
  if (16 * (g0 + t) < n) a.before[g0 + t] = at;
  __syncthreads();
  constexpr int kBatch = 4;
  for (int r = 0; r < kScanItems; r += kBatch) {
    int in[kBatch], out[kBatch], to[kBatch];
    uint8_t pr[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int c = (r + u) * kTileThreads + t;  // cell of the tile
      const uint32_t f = s_m[c >> 4];
      to[u] = (f >> (c & 15)) & 1u ? s_at[c >> 4] + __popc(f & ((1u << (c & 15)) - 1u)) : -1;
      const int64_t cell = 16 * g0 + c;
      if (to[u] >= 0) {
        in[u] = a.inner[cell];
        out[u] = a.outer[cell];
        pr[u] = a.pair[cell];
      }
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      if (to[u] < 0) continue;
      a.out_inner[to[u]] = in[u];
      a.out_outer[to[u]] = out[u];
      a.out_pair[to[u]] = pr[u];
    }
  }
  if (tile == tiles - 1 && t == 0) *a.out_count = found > a.cap ? found : end;
}

// Moves each inner hit's range of cells with them (unless they overflowed), and
// leaves the cells as found in the places of the output past the kept ones.
template <class T>
__global__ void k_fb_ranges(FbArgs<T> a) {
  const int n = stored(a);
  if (n == 0) return;
  auto kept_before = [&](int c) {  // c in [0, n]
    const int g = (c < n ? c : n - 1) >> 4;
    return a.before[g] + __popc(flags16(a, g, n) & ((1u << (c - 16 * g)) - 1u));
  };
  const int first = blockIdx.x * blockDim.x + threadIdx.x, step = gridDim.x * blockDim.x;
  for (int h = first; h < a.n_hits; h += step) {
    const int cnt = a.inner_count[h];
    if (cnt <= 0) continue;
    const int f = a.inner_first[h];
    const int p = kept_before(f);
    a.inner_first[h] = p;
    a.inner_count[h] = kept_before(f + cnt) - p;
  }
  for (int c = kept_before(n) + first; c < n; c += step) {
    a.out_inner[c] = a.inner[c];
    a.out_outer[c] = a.outer[c];
    a.out_pair[c] = a.pair[c];
  }
}

// Workspace after the cells as found and the outer-hit index: flags, lists,
// states.
template <class T>
void carve_rest(Carver& c, FbArgs<T>* a, int cap, int n_hits) {
  const size_t groups = (static_cast<size_t>(cap) + 15) / 16;
  a->keep = c.take<uint8_t>(16 * groups);
  a->before = c.take<int32_t>(groups);
  for (int i = 0; i < kTiers; ++i) a->list[i] = c.take<int32_t>(static_cast<size_t>(n_hits));
  a->n_list = c.take<int32_t>(kTiers);
  a->state_words = static_cast<int32_t>(scan_state_words(cap));
  a->state = c.take<uint64_t>(static_cast<size_t>(a->state_words));
}

// Work-groups of a listed tier's kernel that are resident at once on this
// GPU: its grid is persistent, so more would only queue behind the first ones
// and fewer would leave wavefront slots empty.  Looked up once per device,
// tier and input type, never while a graph is being captured (a plan looks
// it up when it is created); 1024 when unknown.
constexpr int kMaxDevices = 64;
std::mutex g_grid_mu;
int g_listed_grid[kTiers][2][kMaxDevices] = {};

template <class T, int TIER>
int listed_grid() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 1024;
  std::lock_guard<std::mutex> g(g_grid_mu);
  int& v = g_listed_grid[TIER][sizeof(T) == sizeof(double)][dev];
  if (v == 0 && !g_capturing) {
    int cus = 0, per = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_fb_kill<T, TIER>, kTierTeam[TIER], 0) == hipSuccess &&
        cus > 0 && per > 0)
      v = cus * per;
    else
      (void)hipGetLastError();
  }
  return v > 0 ? v : 1024;
}

template <class T>
pt_err run_fishbone(const pt_hits& h, const DevCfg& k, const pt_cells& raw, pt_cells& cells, Carver c, hipStream_t s) {
  const int n_hits = h.n_hits;
  const int cap = cells.cap;
  FbArgs<T> a{};
  a.x = static_cast<const T*>(h.x);
  a.y = static_cast<const T*>(h.y);
  a.z = static_cast<const T*>(h.z);
  a.n_hits = n_hits;
  a.theta2 = k.fishbone_theta2;
  {
    // buckets at least 1% wider than the largest angle of two aligned
    // vectors (plus a margin far above the float rounding of the keys), so
    // that keys within that angle fall in the same or neighbouring buckets
    const double th = std::sqrt(k.fishbone_theta2);
    const double win = th >= 1.0 ? 2.0 : std::asin(th) + 1e-5;
    a.nb = static_cast<int32_t>(std::min<double>(kNB, std::max(1.0, std::floor(2.0 / (win * 1.01)))));
    a.kwin = static_cast<float>(win * 1.001);
    // a unit vector in single precision is within 4e-7 of the true one in
    // each component, so a dot product of two within 1e-6 of the cosine and
    // its square within 2e-6 of the cosine's
    a.cos2_min = th >= 1.0 ? -1.f : static_cast<float>(1.0 - k.fishbone_theta2 - 4e-6);
  }
  a.found = raw.count;
  a.cap = cap;
  a.inner = raw.inner;
  a.outer = raw.outer;
  a.pair = raw.pair;
  a.inner_first = cells.inner_first;
  a.inner_count = cells.inner_count;
  a.out_inner = cells.inner;
  a.out_outer = cells.outer;
  a.out_pair = cells.pair;
  a.out_count = cells.count;
  const pt_err e = build_outer_index(h, raw, c, a.idx, s);
  if (e != PT_OK) return e;
  carve_rest(c, &a, cap, n_hits);
  k_fb_flags<T><<<grid_for(std::max(cap / 16 + 1, a.state_words), kBlock), kBlock, 0, s>>>(a);
  k_fb_kill<T, 0><<<static_cast<unsigned>(n_hits), kTierTeam[0], 0, s>>>(a);
  k_fb_kill<T, 1><<<std::min(n_hits, listed_grid<T, 1>()), kTierTeam[1], 0, s>>>(a);
  k_fb_kill<T, 2><<<std::min(n_hits, listed_grid<T, 2>()), kTierTeam[2], 0, s>>>(a);
  k_fb_kill_big<T><<<256, kBigBlock, 0, s>>>(a);
  PT_LAUNCH_CHECK();
  k_fb_compact<T><<<static_cast<unsigned>(tiles_of(cap, kTileItems)), kTileThreads, 0, s>>>(a);
  k_fb_ranges<T><<<grid_for(std::max(n_hits, cap / 8), kBlock), kBlock, 0, s>>>(a);
  PT_LAUNCH_CHECK();
  return PT_OK;
}

}  // namespace

size_t ws_fishbone(int n_hits, int cells_cap) {
  Carver c(nullptr);
  (void)carve_raw_cells(c, pt_cells{}, cells_cap);
  c.off += ws_outer_index(n_hits, cells_cap);
  FbArgs<float> a{};
  carve_rest(c, &a, cells_cap, n_hits);
  return c.off + 512;
}

pt_cells carve_raw_cells(Carver& c, const pt_cells& cells, int cells_cap) {
  pt_cells raw = cells;
  raw.inner = c.take<int32_t>(static_cast<size_t>(cells_cap));
  raw.outer = c.take<int32_t>(static_cast<size_t>(cells_cap));
  raw.pair = c.take<uint8_t>(static_cast<size_t>(cells_cap));
  raw.count = c.take<int32_t>(1);
  return raw;
}

void fishbone_prepare() {
  (void)listed_grid<float, 1>();
  (void)listed_grid<float, 2>();
  (void)listed_grid<double, 1>();
  (void)listed_grid<double, 2>();
}

pt_err launch_fishbone(const pt_hits& h, const DevCfg& k, const pt_cells& raw, pt_cells& cells, Carver c,
                       hipStream_t s) {
  void* tok = timing_begin(s);
  const pt_err e = h.dtype == PT_F64 ? run_fishbone<double>(h, k, raw, cells, c, s)
                                     : run_fishbone<float>(h, k, raw, cells, c, s);
  timing_end(tok, "fishbone", s);
  return e;
}

}  // namespace pt
