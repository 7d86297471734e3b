// Per-tile work plan: which workgroup takes which tile, built on the device
// from a measured per-tile work count (no host synchronisation).
//
// Paper: Sec. IV (workload imbalance across tiles of dense and sparse
// regions, and adaptive thread-block merging by a density measure).  Here the
// measure is the tile's work count -- its list length before the forward,
// the largest number of entries any of its pixels walks (n_contrib) before the
// backward.  Tiles whose count exceeds kHeavyFactor times the mean are
// *heavy* and are taken first, largest first, so that the longest workgroups
// start at the beginning of the launch instead of forming its tail; tiles
// with at most kLightMax entries are *light* and are merged four to a
// workgroup (one wave per tile, four pixels per lane); the rest keep the
// plain one-workgroup-per-tile form.  Every tile's arithmetic is the same in
// every form, so the image and gradients do not depend on the plan.
//
// Plan layout (int32): [0] heavy count H, [1] medium count M, [2] light count
// L, [3] workgroups needed H + M + ceil(L / 4), then from kPlanHeader the
// tiles: heavy by decreasing count (ties by tile index), medium and light in
// tile order.
#include "gs_internal.h"

namespace gs {

constexpr int kPlanThreads = 1024;
constexpr int kPlanRegs = 16;   // tiles per thread held in registers by k_batch_plan
constexpr int kHeavyCap = 1024;    // at most this many heavy tiles are ordered

// Plan workspace in int32 values for ntiles tiles.
size_t plan_ints(int ntiles) { return kPlanHeader + static_cast<size_t>(ntiles); }

// counts == NULL: a tile's count is its list length from ranges.  Thread t
// owns a contiguous run of tiles, so one block-wide scan of three class
// counts gives every tile its place (tile order inside each class).
__global__ __launch_bounds__(kPlanThreads) void k_tile_plan(int ntiles, const uint2* __restrict__ ranges,
                                                            const uint32_t* __restrict__ counts,
                                                            float heavy_factor, int light_max,
                                                            int32_t* __restrict__ plan) {
  __shared__ float s_red[kPlanThreads / 64];
  __shared__ uint32_t s_scan[3][kPlanThreads / 64];
  __shared__ uint32_t s_hw[kHeavyCap];
  __shared__ int s_ht[kHeavyCap];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int32_t* const order = plan + kPlanHeader;
  auto count_of = [&](int t) -> uint32_t { return counts ? counts[t] : (ranges[t].y - ranges[t].x); };
  const int per = (ntiles + kPlanThreads - 1) / kPlanThreads;
  const int t0 = min(ntiles, tid * per), t1 = min(ntiles, t0 + per);

  float sum = 0.f;
  for (int t = t0; t < t1; ++t) sum += static_cast<float>(count_of(t));
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
  if (lane == 0) s_red[wave] = sum;
  __syncthreads();
  float total = 0.f;
  for (int w = 0; w < kPlanThreads / 64; ++w) total += s_red[w];
  const float thresh = fmaxf(heavy_factor * total / static_cast<float>(max(ntiles, 1)),
                             static_cast<float>(light_max));
  auto cls_of = [&](uint32_t w) -> int {
    return static_cast<float>(w) > thresh ? 0 : (static_cast<int>(w) <= light_max ? 2 : 1);
  };
  // per-thread class counts, then an exclusive scan over threads (wave
  // shuffles, then the wave totals in LDS)
  uint32_t c[3] = {0u, 0u, 0u};
  for (int t = t0; t < t1; ++t) ++c[cls_of(count_of(t))];
  uint32_t ex[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    uint32_t incl = c[k];
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t v = __shfl_up(incl, o, 64);
      if (lane >= o) incl += v;
    }
    ex[k] = incl - c[k];
    if (lane == 63) s_scan[k][wave] = incl;
  }
  __syncthreads();
  uint32_t tot[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    uint32_t before = 0, all = 0;
    for (int w = 0; w < kPlanThreads / 64; ++w) {
      const uint32_t v = s_scan[k][w];
      before += (w < wave) ? v : 0u;
      all += v;
    }
    ex[k] += before;
    tot[k] = all;
  }
  const int H = static_cast<int>(min(tot[0], static_cast<uint32_t>(kHeavyCap)));
  const int O = static_cast<int>(tot[0]) - H;          // heavy beyond the cap: placed after the medium ones
  const int M = static_cast<int>(tot[1]), L = static_cast<int>(tot[2]);
  for (int t = t0; t < t1; ++t) {
    const uint32_t w = count_of(t);
    const int k = cls_of(w);
    const int pos = static_cast<int>(ex[k]++);
    if (k == 0) {
      if (pos < kHeavyCap) { s_hw[pos] = w; s_ht[pos] = t; }
      else order[H + M + (pos - kHeavyCap)] = t;
    } else if (k == 1) {
      order[H + pos] = t;
    } else {
      order[H + M + O + pos] = t;
    }
  }
  __syncthreads();
  // heavy tiles: rank by (count descending, tile ascending)
  for (int i = tid; i < H; i += kPlanThreads) {
    const uint32_t wi = s_hw[i];
    const int ti = s_ht[i];
    int r = 0;
    for (int j = 0; j < H; ++j) {
      const uint32_t wj = s_hw[j];
      r += (wj > wi || (wj == wi && s_ht[j] < ti)) ? 1 : 0;
    }
    order[r] = ti;
  }
  if (tid == 0) {
    plan[0] = H;
    plan[1] = M + O;
    plan[2] = L;
    plan[3] = H + M + O + (L + 3) / 4;
  }
}

// Backward work items: every batch of 256 list entries that some pixel of
// the tile walks becomes its own workgroup, (tile, batch) in tile order.  A
// tile's walk length is min(list length, largest n_contrib) -- the counts the
// forward left in `work`, four per tile.  Tiles with a count of at most
// light_max go to the light list instead (a plan with H = M = 0), or nowhere
// when light is NULL (with light_max = 0: the tiles whose pixels blend
// nothing).
// items: [0] item count, from kPlanHeader four ints per item: the tile, the
// batch, the tile's first list position and its walk length (so that the
// workgroup's list loads wait for nothing else).
// The first ceil(ntiles / 1024) workgroups build the plan, 1,024 tiles each:
// every one adds up the batches of all tiles before its own itself (24 bytes
// per tile, read from L2; one workgroup writing every item took 22.5 us against
// 17.3 for 6,700 tiles and 1M rows to clear).  The others, if any, clear
// zero[0, zero_n4) meanwhile (the backward's accumulator rows).

// Sums over the workgroup of two values per thread (s_w: two words per wave,
// free again on return).
__device__ __forceinline__ void block_sum2(uint32_t& a, uint32_t& b, uint32_t (*s_w)[2]) {
  for (int o = 32; o > 0; o >>= 1) {
    a += __shfl_xor(a, o, 64);
    b += __shfl_xor(b, o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    s_w[threadIdx.x >> 6][0] = a;
    s_w[threadIdx.x >> 6][1] = b;
  }
  __syncthreads();
  a = b = 0u;
  for (int w = 0; w < kPlanThreads / 64; ++w) {
    a += s_w[w][0];
    b += s_w[w][1];
  }
  __syncthreads();
}
// Exclusive prefixes over the workgroup of two values per thread.
__device__ __forceinline__ void block_prefix2(uint32_t& a, uint32_t& b, uint32_t (*s_w)[2]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t ia = a, ib = b;
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t u = __shfl_up(ia, o, 64), v = __shfl_up(ib, o, 64);
    if (lane >= o) { ia += u; ib += v; }
  }
  if (lane == 63) { s_w[wave][0] = ia; s_w[wave][1] = ib; }
  __syncthreads();
  a = ia - a;
  b = ib - b;
  for (int w = 0; w < wave; ++w) {
    a += s_w[w][0];
    b += s_w[w][1];
  }
  __syncthreads();
}

__global__ __launch_bounds__(kPlanThreads) void k_batch_plan(int ntiles, const uint2* __restrict__ ranges,
                                                             const uint32_t* __restrict__ work, int light_max,
                                                             int32_t* __restrict__ items,
                                                             int32_t* __restrict__ light,
                                                             float4* __restrict__ zero, int64_t zero_n4) {
  const int plans = (ntiles + kPlanThreads - 1) / kPlanThreads;
  if (static_cast<int>(blockIdx.x) >= plans) {
    const int64_t stride = static_cast<int64_t>(gridDim.x - plans) * kPlanThreads;
    for (int64_t i = static_cast<int64_t>(blockIdx.x - plans) * kPlanThreads + threadIdx.x; i < zero_n4; i += stride)
      zero[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    return;
  }
  __shared__ uint32_t s_w[kPlanThreads / 64][2];
  const int tid = threadIdx.x, first = blockIdx.x * kPlanThreads;
  // a tile's first list position, walk length (0: no items) and whether it is light
  struct Walk {
    uint32_t first, len;
    bool light;
  };
  auto walk_at = [&](int t) -> Walk {
    const uint2 rg = t < ntiles ? ranges[t] : make_uint2(0u, 0u);
    const uint32_t wk = t < ntiles ? tile_work_of(work, t) : 0u;
    const bool small = static_cast<int>(wk) <= light_max;
    return Walk{rg.x, small ? 0u : min(rg.y - rg.x, wk), small && wk > 0u};
  };
  auto batches = [](uint32_t len) -> uint32_t { return (len + 255u) / 256u; };
  // items and light tiles before this workgroup's; up to kPlanRegs tiles per
  // thread have all their loads in flight together
  uint32_t at = 0u, lat = 0u;
  auto count = [&](const Walk& w) {
    at += batches(w.len);
    lat += w.light ? 1u : 0u;
  };
  const int before = static_cast<int>(blockIdx.x);
  if (before <= kPlanRegs) {
    Walk w[kPlanRegs];
#pragma unroll
    for (int k = 0; k < kPlanRegs; ++k) w[k] = k < before ? walk_at(k * kPlanThreads + tid) : Walk{0u, 0u, false};
#pragma unroll
    for (int k = 0; k < kPlanRegs; ++k) count(w[k]);
  } else {
    for (int k = 0; k < before; ++k) count(walk_at(k * kPlanThreads + tid));
  }
  const Walk own = walk_at(first + tid);
  const uint32_t n = batches(own.len);
  block_sum2(at, lat, s_w);
  uint32_t pa = n, pl = own.light ? 1u : 0u;
  block_prefix2(pa, pl, s_w);
  at += pa;
  lat += pl;
  int4* const out = reinterpret_cast<int4*>(items + kPlanHeader);   // items is 16-byte aligned
  for (uint32_t b = 0; b < n; ++b)
    out[at + b] = make_int4(first + tid, static_cast<int>(b), static_cast<int>(own.first), static_cast<int>(own.len));
  if (light && own.light) light[kPlanHeader + lat] = first + tid;
  // the last tile's thread knows the totals
  if (first + tid == ntiles - 1) {
    items[0] = static_cast<int32_t>(at + n);
    if (light) { light[0] = 0; light[1] = 0; light[2] = static_cast<int32_t>(lat + (own.light ? 1u : 0u)); light[3] = 0; }
  }
}

gs_status launch_batch_plan(int ntiles, const uint32_t* ranges, const uint32_t* work, int light_max, int32_t* items,
                            int32_t* light, float4* zero, int64_t zero_n4, hipStream_t s) {
  const unsigned fill = zero_n4 > 0 ? static_cast<unsigned>(std::min<int64_t>(ceil_div(zero_n4, kPlanThreads), 1024)) : 0u;
  { TimedLaunch gs_tl("k_batch_plan", s); k_batch_plan<<<static_cast<unsigned>(ceil_div(ntiles, kPlanThreads)) + fill, kPlanThreads, 0, s>>>(ntiles, reinterpret_cast<const uint2*>(ranges), work, light_max, items,
                                          light, zero, zero_n4); }
  return check_launch("k_batch_plan");
}

gs_status launch_tile_plan(int ntiles, const uint32_t* ranges, const uint32_t* counts, float heavy_factor,
                           int light_max, int32_t* plan, hipStream_t s) {
  { TimedLaunch gs_tl("k_tile_plan", s); k_tile_plan<<<1, kPlanThreads, 0, s>>>(ntiles, reinterpret_cast<const uint2*>(ranges), counts, heavy_factor,
                                         light_max, plan); }
  return check_launch("k_tile_plan");
}

}  // namespace gs
