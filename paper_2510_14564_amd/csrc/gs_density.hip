// Workload-sensitive density control (Sec. III-C): each point's local density
// (other points within a radius r), the statistical thresholds mu -/+ sigma of
// the densities, the mean distance to the k nearest points, one round of
// densification next to sparse points (Gaussian spread a d_bar plus a uniform
// perturbation, from noise the caller draws) and the merging of mutual
// nearest dense pairs within mu_d + gamma sigma_d.
//
// The neighbour searches run on a uniform grid of cells of side h = 1.07 r,
// counting-sorted by bucket (one pass of atomics, whose returned values are
// the ranks, then the library's exclusive scan).  A row of cells along x
// starts at a hash of its (y, z) in a power-of-two table and its cells follow
// one another there, so the cells x - R .. x + R of a row are one contiguous
// run of points and a search over (2R + 1)^3 cells reads (2R + 1)^2 runs.
// A point's cell is floor(x / h) per axis in FP32; with every coordinate below
// 2^18 h in magnitude the FP32 cell coordinates of two points differ from
// their exact value by less than 1/16 of a cell, so a point within r of
// another lies in the same or an adjacent cell (27 cells cover the radius
// search), and after the cells up to Chebyshev offset R have been scanned
// every point closer than (R - 1/16) h has been seen (the k-nearest search
// stops on that guarantee).  One pass over the 27 cells, four lanes per query,
// gives a query's density and the k nearest of them; a query whose k-th nearest
// lies farther (one in seven at a 100x density skew with 20 neighbours in r)
// goes on to half a wave that scans R = 2 and 3, one in fifty of those to a
// workgroup that scans R = 7, and the few left after that to workgroups that
// scan every point.
// Rows can share buckets; where two runs of a search share one, only the points
// whose own row is the run's count (a row's run holds each of its points once),
// so nothing is counted twice.
//
// Every decision is taken exactly as the definition states it in the
// precision it names: FP32 squared distances (each operation rounded, no
// fused multiply-add), thresholds in FP64 from exact integer sums with
// correctly rounded operations, nearest points by (FP32 squared distance,
// index).  This file is compiled without contraction of products into fused
// multiply-adds; sqrt and division are IEEE-rounded (HIP's default for FP32
// square roots and quotients in source), so the square-root sums are the
// definition's too.  The densities, classes, neighbour lists and the merge pairing are
// therefore the definition's bit for bit; the new and merged parameters are
// FP32 evaluations of their formulas.
#include "gs_internal.h"

namespace gs {

constexpr float kDcCellScale = 1.07f;
constexpr int kDcLanes = 4;         // lanes per query of the search over 27 cells (4 or 8)
constexpr uint32_t kDcSlots = 64;    // slots of the statistics' sums (one per lane of the wave that adds them up)

__device__ __forceinline__ float dc_floor(float x, float inv_h) { return floorf(__fmul_rn(x, inv_h)); }

// Position of cell (0, cy, cz) in the table; the row's cell cx lies cx further on, modulo the table.
__device__ __forceinline__ uint32_t dc_row(int cy, int cz) {
  uint32_t h = static_cast<uint32_t>(cy) * 19349663u ^ static_cast<uint32_t>(cz) * 83492791u;
  h ^= h >> 15;
  h *= 0x2c1b3c6du;
  return h ^ h >> 12;
}

// FP32 squared distance from the query q to point p, rounded step by step.
__device__ __forceinline__ float dc_d2(const float4& q, const float4& p) {
  const float dx = __fsub_rn(q.x, p.x), dy = __fsub_rn(q.y, p.y), dz = __fsub_rn(q.z, p.z);
  float s = __fmul_rn(dx, dx);
  s = __fadd_rn(s, __fmul_rn(dy, dy));
  return __fadd_rn(s, __fmul_rn(dz, dz));
}

// The far search splits each remaining query's scan over every point into S
// ranges, one workgroup each, while count * S fits kFarSlots partial lists
// (S = min(64, kFarSlots / count)); beyond that, one workgroup per query
// scans all points and writes the result itself.
constexpr uint32_t kFarSlots = 16384;
constexpr uint32_t kFarSplitMax = 64;
__host__ __device__ __forceinline__ uint32_t far_splits(uint32_t count) {
  return count == 0 || count > kFarSlots ? 1u : (kFarSlots / count < kFarSplitMax ? kFarSlots / count : kFarSplitMax);
}

struct DcSums {            // one slot of the statistics' sums, a cache line of its own
  unsigned long long c1, c2;  // rho, rho^2
  double a1, a2;              // nearest distance, its square
  unsigned long long pad[4];
};

struct DcReport {          // what the host reads back, in one copy
  double stat[8];          // mu, sigma, rho_low, rho_high, mu_d, sigma_d, d_merge, unused
  unsigned long long total;   // kept + new (from the scan)
  uint32_t kept;
  uint32_t range;          // set if a coordinate is out of the cells' range
};

struct DcWs {
  uint32_t* count;      // [T] points per bucket, then their exclusive prefix (bucket starts)
  uint32_t* scan;       // scan block sums
  float4* pts;          // [n] x, y, z, index (bits) in bucket order
  uint2* cell;          // [n] each point's bucket and rank in it
  int32_t* rho;         // [n]
  int32_t* nn;          // [n] nearest other point
  float* dnn;           // [n] its distance
  float* dbar;          // [n] mean distance to the k nearest
  uint32_t* pos;        // [2n] 1 if the point survives, then 1 if it spawns a new one; then their exclusive prefix,
                        // which is the output position of each
  int32_t* partner;     // [n] merge partner or -1
  DcSums* sums;         // [kDcSlots]
  DcReport* rep;        // [1]
  uint32_t* far;        // [n] queries the 27 cells left, [1] their count (far_n)
  uint32_t* far_n;
  uint32_t* far2;       // [n] queries the half waves left, [1] their count
  uint32_t* far2_n;
  uint32_t* far3_n;     // [1] count of the queries the workgroups left (they take the place of far's)
  double* cand;         // [kFarSlots][8] partial k-nearest lists of the split far search
  size_t bytes;
};

static uint32_t dc_table(int64_t n) {
  uint32_t t = 1024;
  while (static_cast<int64_t>(t) < 2 * n && t < (1u << 30)) t <<= 1;
  return t;
}

static DcWs carve_dc(void* base, int64_t n) {
  Carver c(base);
  DcWs w;
  const uint32_t T = dc_table(n);
  const size_t nn = static_cast<size_t>(std::max<int64_t>(n, 1));
  w.count = c.take<uint32_t>(T);
  w.scan = c.take<uint32_t>(std::max(scan_sums_words(T), scan_sums_words(2 * n)));
  w.pts = c.take<float4>(nn);
  w.cell = c.take<uint2>(nn);
  w.rho = c.take<int32_t>(nn);
  w.nn = c.take<int32_t>(nn);
  w.dnn = c.take<float>(nn);
  w.dbar = c.take<float>(nn);
  w.pos = c.take<uint32_t>(2 * nn);
  w.partner = c.take<int32_t>(nn);
  w.sums = c.take<DcSums>(kDcSlots);
  w.rep = c.take<DcReport>(1);
  w.far = c.take<uint32_t>(nn);
  w.far_n = c.take<uint32_t>(1);
  w.far2 = c.take<uint32_t>(nn);
  w.far2_n = c.take<uint32_t>(1);
  w.far3_n = c.take<uint32_t>(1);
  w.cand = c.take<double>(static_cast<size_t>(kFarSlots) * 8);
  w.bytes = c.off;
  return w;
}

size_t density_workspace(int64_t n) { return carve_dc(nullptr, n).bytes; }

__global__ __launch_bounds__(256) void k_dc_clear(uint32_t* __restrict__ count, uint32_t T, DcSums* __restrict__ sums,
                                                  DcReport* __restrict__ rep, uint32_t* __restrict__ far_n,
                                                  uint32_t* __restrict__ far2_n, uint32_t* __restrict__ far3_n) {
  const uint32_t i = blockIdx.x * 256 + threadIdx.x;
  if (i < T) count[i] = 0u;
  if (i < kDcSlots) sums[i] = DcSums{};
  if (i == 0) {
    *rep = DcReport{};
    far_n[0] = 0u; far2_n[0] = 0u; far3_n[0] = 0u;
  }
}

// Each point's bucket and its rank there (the bucket's count when it came).  A
// coordinate of 2^18 cells or more (or not finite) sets the report's range
// flag: the cell guarantees above need |x| < 2^18 h.
__global__ __launch_bounds__(256) void k_dc_cells(int n, const float* __restrict__ means, float inv_h, uint32_t mask,
                                                  uint2* __restrict__ cell, uint32_t* __restrict__ count,
                                                  DcReport* __restrict__ rep) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const float x = means[i], y = means[static_cast<int64_t>(n) + i], z = means[2 * static_cast<int64_t>(n) + i];
  const float lim = 262144.0f;
  uint32_t b = 0u;
  if (fabsf(__fmul_rn(x, inv_h)) < lim && fabsf(__fmul_rn(y, inv_h)) < lim && fabsf(__fmul_rn(z, inv_h)) < lim) {
    b = (dc_row(static_cast<int>(dc_floor(y, inv_h)), static_cast<int>(dc_floor(z, inv_h))) +
         static_cast<uint32_t>(static_cast<int>(dc_floor(x, inv_h)))) & mask;
  } else {
    atomicOr(&rep->range, 1u);
  }
  cell[i] = make_uint2(b, atomicAdd(&count[b], 1u));
}

__global__ __launch_bounds__(256) void k_dc_scatter(int n, const float* __restrict__ means,
                                                    const uint2* __restrict__ cell, const uint32_t* __restrict__ start,
                                                    float4* __restrict__ pts) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const uint2 c = cell[i];
  pts[start[c.x] + c.y] =
      make_float4(means[i], means[static_cast<int64_t>(n) + i], means[2 * static_cast<int64_t>(n) + i], __int_as_float(i));
}

// A candidate as one ordered value: the FP32 squared distance's bits above the
// index, read as a double.  Both parts are non-negative, so doubles compare as
// (distance, index) does, and keeping the K best sorted is 2K - 1 minima and
// maxima with no branch.  An empty slot holds 3.0e38; everything above it -- an
// overflowed distance, or the NaN that stands for no candidate -- never
// displaces one.
__device__ __forceinline__ double dc_key(float d2, int i) { return __hiloint2double(__float_as_int(d2), i); }
__device__ __forceinline__ double dc_empty() { return dc_key(3.0e38f, 0x7fffffff); }
__device__ __forceinline__ float dc_none() { return __int_as_float(0x7fc00000); }
__device__ __forceinline__ float dc_key_d2(double k) { return __int_as_float(__double2hiint(k)); }

template <int K>
__device__ __forceinline__ void dc_insert(double (&b)[K], double c) {
#pragma unroll
  for (int m = 0; m < K; ++m) {
    const double lo = __builtin_fmin(b[m], c);
    c = __builtin_fmax(b[m], c);
    b[m] = lo;
  }
}

// The value of the lane that a DPP control names.
template <int CTRL>
__device__ __forceinline__ double dc_dpp(double v) {
  return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true),
                          __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true));
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140;

template <int K, int CTRL>
__device__ __forceinline__ void dc_merge_dpp(double (&b)[K]) {
  double o[K];
#pragma unroll
  for (int m = 0; m < K; ++m) o[m] = dc_dpp<CTRL>(b[m]);
#pragma unroll
  for (int m = 0; m < K; ++m) dc_insert<K>(b, o[m]);
}

template <int K>
__device__ __forceinline__ void dc_merge_shfl(double (&b)[K], int off) {
  double o[K];
#pragma unroll
  for (int m = 0; m < K; ++m) o[m] = __shfl_xor(b[m], off, 64);
#pragma unroll
  for (int m = 0; m < K; ++m) dc_insert<K>(b, o[m]);
}

// The K best of 8 lanes' lists, in each of the 8.  (After the first two steps
// the four lanes of a quad hold the same list, so the mirror of the eight
// brings the other quad's.)
template <int K>
__device__ __forceinline__ void dc_merge8(double (&b)[K]) {
  dc_merge_dpp<K, kDppXor1>(b);
  dc_merge_dpp<K, kDppXor2>(b);
  dc_merge_dpp<K, kDppHalfMirror>(b);
}

template <int K>
__device__ __forceinline__ void dc_merge64(double (&b)[K]) {
  dc_merge8<K>(b);
  dc_merge_dpp<K, kDppMirror>(b);
  dc_merge_shfl<K>(b, 16);
  dc_merge_shfl<K>(b, 32);
}

// A query's results from its K best: nearest point, its distance and the mean
// distance of the keff nearest (FP32: square roots summed in order, over
// keff).  Returns the nearest distance.
template <int K>
__device__ __forceinline__ float dc_finish(const double (&b)[K], int keff, int qi, int32_t* __restrict__ nn,
                                           float* __restrict__ dnn, float* __restrict__ dbar) {
  float sum = 0.0f;
#pragma unroll
  for (int m = 0; m < K; ++m)
    if (m < keff) sum = __fadd_rn(sum, sqrtf(dc_key_d2(b[m])));
  const float d0 = keff > 0 ? sqrtf(dc_key_d2(b[0])) : 0.0f;
  nn[qi] = keff > 0 ? __double2loint(b[0]) : -1;
  dnn[qi] = d0;
  dbar[qi] = keff > 0 ? sum / static_cast<float>(keff) : 0.0f;
  return d0;
}

// A workgroup's share of the statistics into a slot: one set of atomics per
// workgroup, spread over kDcSlots lines (the first wave; lane t has a query's
// density and nearest distance, or zeros).
__device__ __forceinline__ void dc_add_sums(int cnt, float d0, DcSums* __restrict__ sums) {
  unsigned long long c1 = static_cast<unsigned long long>(cnt), c2 = c1 * c1;
  double a1 = static_cast<double>(d0), a2 = a1 * a1;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    c1 += __shfl_xor(c1, o, 64);
    c2 += __shfl_xor(c2, o, 64);
    a1 += __shfl_xor(a1, o, 64);
    a2 += __shfl_xor(a2, o, 64);
  }
  if (threadIdx.x == 0) {
    DcSums* d = sums + blockIdx.x % kDcSlots;
    if (c2) {
      atomicAdd(&d->c1, c1);
      atomicAdd(&d->c2, c2);
    }
    if (a2 != 0.0) {
      unsafeAtomicAdd(&d->a1, a1);
      unsafeAtomicAdd(&d->a2, a2);
    }
  }
}

// The first bucket of the cells cx - R .. cx + R of row (cy, cz).
__device__ __forceinline__ uint32_t dc_bucket(uint32_t T, int cx, int cy, int cz, int R) {
  return (dc_row(cy, cz) + static_cast<uint32_t>(cx - R)) & (T - 1u);
}

// Points [x, y) in bucket order of the 2R + 1 < T buckets from b0; where they
// wrap round the table y exceeds n, and position p >= n is p - n.
__device__ __forceinline__ uint2 dc_run(const uint32_t* __restrict__ start, uint32_t T, int n, uint32_t b0, int R) {
  const uint32_t mask = T - 1u;
  const uint32_t b1 = (b0 + 2u * static_cast<uint32_t>(R)) & mask;
  const uint32_t s = start[b0];
  const uint32_t e = b1 < mask ? start[b1 + 1u] : static_cast<uint32_t>(n);
  return make_uint2(s, b1 < b0 ? e + static_cast<uint32_t>(n) : e);
}

__device__ __forceinline__ void dc_wave_sync() {   // a wave's own LDS writes are visible to its lanes
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ float4 dc_at(const float4* __restrict__ pts, uint32_t p, int n) {
  return pts[min(p, p - static_cast<uint32_t>(n))];
}

// Densities and near neighbours, G lanes per query over the nine runs of its 27
// cells: rho = other points within r, the sums of rho and rho^2, and where the
// K nearest lie inside the 27 cells' guarantee the K-nearest results (a query
// left goes to the wave kernel).
//
// As long as no two of a query's runs share a bucket, each point comes up at
// most once whatever rows share its bucket, and a point of another row is only
// one more point whose distance is looked at; so a candidate's own row is
// looked at only by waves of which a query has overlapping runs (36 pairs,
// 5/T each), or one that wraps round the table.
// Instruction issue bounds it (30 VALU instructions a candidate, 171 candidates
// a query, three quarters of the lanes busy): 64 us at 200,000 points, radius
// 0.03.  One thread per query over hashed cells, density and neighbours apart,
// took 341 + 810 us; with the row looked at for every candidate, 133.  Eight lanes
// per query take the same time and more registers.
template <int K>
__global__ __launch_bounds__(256) void k_dc_near(int n, const float4* __restrict__ pts,
                                                 const uint32_t* __restrict__ start, uint32_t T, float h, float inv_h,
                                                 float r2, int32_t* __restrict__ rho, int32_t* __restrict__ nn,
                                                 float* __restrict__ dnn, float* __restrict__ dbar,
                                                 DcSums* __restrict__ sums, uint32_t* __restrict__ far,
                                                 uint32_t* __restrict__ far_n) {
  constexpr int G = kDcLanes, kHeld = (9 + G - 1) / G;   // runs that a lane looks up: l, l + G, ..
  __shared__ int s_cnt[256 / G];
  __shared__ float s_d0[256 / G];
  const int l = threadIdx.x & (G - 1), group = threadIdx.x / G;
  const int s = blockIdx.x * (256 / G) + group;
  const bool live = s < n;
  const float4 q = pts[live ? s : n - 1];
  const int qi = __float_as_int(q.w);
  const float fy = dc_floor(q.y, inv_h), fz = dc_floor(q.z, inv_h);
  const int cx = static_cast<int>(dc_floor(q.x, inv_h)), cy = static_cast<int>(fy), cz = static_cast<int>(fz);
  // run r = 3 (dz + 1) + dy + 1, its first bucket and its points
  uint32_t b0[kHeld];
  uint2 run[kHeld];
#pragma unroll
  for (int k = 0; k < kHeld; ++k) {
    const int r = min(l + k * G, 8);
    b0[k] = dc_bucket(T, cx, cy + r % 3 - 1, cz + r / 3 - 1, 1);
    run[k] = dc_run(start, T, n, b0[k], 1);
  }
  bool shared = false;
#pragma unroll
  for (int k = 0; k < kHeld; ++k) {
    shared |= run[k].y > static_cast<uint32_t>(n);
    if (!live) run[k].y = run[k].x;
  }
#pragma unroll
  for (int r = 0; r < 9; ++r) {
    const uint32_t o = __shfl(b0[r / G], (threadIdx.x & (64 - G)) | (r % G), 64);
#pragma unroll
    for (int k = 0; k < kHeld; ++k) shared |= ((b0[k] - o + 2u) & (T - 1u)) <= 4u && min(l + k * G, 8) != r;
  }
  double b[K];
#pragma unroll
  for (int m = 0; m < K; ++m) b[m] = dc_empty();
  int cnt = 0;   // the query itself is counted too
  if (!__any(shared)) {
    // a candidate is loaded while the one before it is looked at, a run's first while the run before is
    const uint32_t top = static_cast<uint32_t>(n) - 1u;
    uint32_t p = __shfl(run[0].x, threadIdx.x & (64 - G), 64) + l;
    float4 o = pts[min(p, top)];
#pragma unroll
    for (int r = 0; r < 9; ++r) {
      const uint32_t p1 = __shfl(run[r / G].y, (threadIdx.x & (64 - G)) | (r % G), 64);
      uint32_t q0 = 0;
      float4 o0 = o;
      if (r < 8) {
        q0 = __shfl(run[(r + 1) / G].x, (threadIdx.x & (64 - G)) | ((r + 1) % G), 64) + l;
        o0 = pts[min(q0, top)];
      }
      while (p < p1) {
        p += G;
        const float4 o1 = pts[min(p, top)];
        const int oi = __float_as_int(o.w);
        const float d2 = dc_d2(q, o);
        cnt += d2 <= r2 ? 1 : 0;
        dc_insert<K>(b, dc_key(oi != qi ? d2 : dc_none(), oi));
        o = o1;
      }
      p = q0;
      o = o0;
    }
  } else {
    for (int r = 0; r < 9; ++r) {
      uint2 v = run[0];
#pragma unroll
      for (int k = 1; k < kHeld; ++k) v = r / G == k ? run[k] : v;
      const int src = (threadIdx.x & (64 - G)) | (r % G);
      const uint32_t p1 = __shfl(v.y, src, 64);
      const float wy = fy + static_cast<float>(r % 3 - 1), wz = fz + static_cast<float>(r / 3 - 1);
      for (uint32_t p = __shfl(v.x, src, 64) + l; p < p1; p += G) {
        const float4 o = dc_at(pts, p, n);
        const int oi = __float_as_int(o.w);
        const float d2 = dc_floor(o.y, inv_h) == wy && dc_floor(o.z, inv_h) == wz ? dc_d2(q, o) : dc_none();
        cnt += d2 <= r2 ? 1 : 0;
        dc_insert<K>(b, dc_key(oi != qi ? d2 : dc_none(), oi));
      }
    }
  }
  dc_merge_dpp<K, kDppXor1>(b);
  cnt += __builtin_amdgcn_mov_dpp(cnt, kDppXor1, 0xf, 0xf, true);
  dc_merge_dpp<K, kDppXor2>(b);
  cnt += __builtin_amdgcn_mov_dpp(cnt, kDppXor2, 0xf, 0xf, true);
  if (G == 8) {
    dc_merge_dpp<K, kDppHalfMirror>(b);
    cnt += __builtin_amdgcn_mov_dpp(cnt, kDppHalfMirror, 0xf, 0xf, true);
  }
  cnt -= 1;   // the query itself
  // every point closer than (1 - 1/16) h has been seen
  const float g = 0.9375f * h;
  const bool first = live && l == 0;
  const bool done = n - 1 >= K && dc_key_d2(b[K - 1]) <= g * g * 0.9999f;
  if (first) {
    rho[qi] = cnt;
    s_cnt[group] = cnt;
    s_d0[group] = done ? dc_finish<K>(b, K, qi, nn, dnn, dbar) : -1.0f;
  }
  // one append per workgroup: one per wave, 16 queries, was 35 us of 103 at 200,000 points
  __syncthreads();
  if (threadIdx.x >= 64) return;
  const int t = threadIdx.x, s0 = blockIdx.x * (256 / G);
  const bool here = t < 256 / G && s0 + t < n;
  const float d0 = here ? s_d0[t] : 0.0f;
  const uint64_t open = __ballot(d0 < 0.0f);
  if (open) {
    uint32_t at = 0;
    if (t == 0) at = atomicAdd(far_n, static_cast<uint32_t>(__popcll(open)));
    at = __builtin_amdgcn_readfirstlane(at);
    if (d0 < 0.0f) far[at + __popcll(open & ((1ull << t) - 1ull))] = static_cast<uint32_t>(s0 + t);
  }
  dc_add_sums(here ? s_cnt[t] : 0, d0 < 0.0f ? 0.0f : d0, sums);
}

// The K nearest among the cells up to R of a query, found by LANES lanes (half a
// wave, or a workgroup; each lane ends with the K best): the lanes look the
// (2R + 1)^2 runs up, and then share all of their points evenly; the runs' ends,
// added up in LDS, tell a lane which run its next point is in.  Returns whether
// they lie inside R's guarantee.
template <int K, int R, int LANES>
__device__ __forceinline__ bool dc_search(double (&b)[K], int n, const float4* __restrict__ pts,
                                          const uint32_t* __restrict__ start, uint32_t T, float h, float inv_h,
                                          const float4& q, uint32_t* __restrict__ end, uint32_t* __restrict__ at,
                                          double* __restrict__ lists) {
  constexpr int kSide = 2 * R + 1, kRuns = kSide * kSide, kWave = LANES < 64 ? LANES : 64;
  const int lane = threadIdx.x & (LANES - 1);
  const float fy = dc_floor(q.y, inv_h), fz = dc_floor(q.z, inv_h);
  const int cx = static_cast<int>(dc_floor(q.x, inv_h)), cy = static_cast<int>(fy), cz = static_cast<int>(fz);
  const int qi = __float_as_int(q.w);
  auto sync = [] {
    if (LANES > 64) __syncthreads();
    else dc_wave_sync();
  };
  uint32_t total = 0;
  sync();   // the search before has read the LDS
#pragma unroll
  for (int t0 = 0; t0 < kRuns; t0 += LANES) {
    const int t = t0 + lane;
    uint2 run = make_uint2(0u, 0u);
    if (t < kRuns) run = dc_run(start, T, n, dc_bucket(T, cx, cy + t % kSide - R, cz + t / kSide - R, R), R);
    const uint32_t len = run.y - run.x;
    uint32_t sum = len;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const uint32_t v = __shfl_up(sum, o, kWave);
      sum += (lane & (kWave - 1)) >= o ? v : 0u;
    }
    if (LANES > 64) {
      if ((lane & 63) == 63) at[lane >> 6] = sum;
      __syncthreads();
      uint32_t before = 0, all = 0;
#pragma unroll
      for (int w = 0; w < LANES / 64; ++w) {
        before += w < lane >> 6 ? at[w] : 0u;
        all += at[w];
      }
      __syncthreads();
      sum += before;
      end[t] = sum;
      at[t] = run.x - (sum - len);
      total = all;
    } else {
      end[t] = total + sum;                   // points of the runs up to this one
      at[t] = run.x - (total + sum - len);    // its first point less the points before it
      total += __shfl(sum, kWave - 1, kWave);
    }
  }
  sync();
#pragma unroll
  for (int m = 0; m < K; ++m) b[m] = dc_empty();
  for (uint32_t c0 = lane; c0 < total; c0 += 2 * LANES) {
    // two points at a time: the search for a point's run is a chain of LDS reads
    float4 o[2];
    int u[2] = {0, 0};   // the run that holds the point: the number of runs that end at or before it
    uint32_t c[2] = {c0, min(c0 + LANES, total - 1u)};
#pragma unroll
    for (int step = kRuns < 32 ? 16 : (kRuns < 64 ? 32 : 128); step > 0; step >>= 1)
#pragma unroll
      for (int i = 0; i < 2; ++i)
        if (end[min(u[i] + step, kRuns) - 1] <= c[i]) u[i] += step;
#pragma unroll
    for (int i = 0; i < 2; ++i) o[i] = dc_at(pts, at[u[i]] + c[i], n);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int oi = __float_as_int(o[i].w);
      const bool in = dc_floor(o[i].y, inv_h) == fy + static_cast<float>(u[i] % kSide - R) &&
                      dc_floor(o[i].z, inv_h) == fz + static_cast<float>(u[i] / kSide - R) && oi != qi &&
                      c0 + i * LANES < total;
      dc_insert<K>(b, dc_key(in ? dc_d2(q, o[i]) : dc_none(), oi));
    }
  }
  dc_merge8<K>(b);
  dc_merge_dpp<K, kDppMirror>(b);
  dc_merge_shfl<K>(b, 16);
  if (LANES > 64) {
    dc_merge_shfl<K>(b, 32);
    if ((lane & 63) == 0) {
#pragma unroll
      for (int m = 0; m < K; ++m) lists[(lane >> 6) * K + m] = b[m];
    }
    __syncthreads();
    for (int w = 0; w < LANES / 64; ++w)
      if (w != lane >> 6)
        for (int m = 0; m < K; ++m) dc_insert<K>(b, lists[w * K + m]);
  }
  const float g = (static_cast<float>(R) - 0.0625f) * h;
  return dc_key_d2(b[K - 1]) <= g * g * 0.9999f;
}

// Queries the 27 cells left, half a wave each: the cells up to R = 2, where nine
// in ten end, then 3; the one in fifty that is left goes on to a workgroup.  (A run
// per lane, with which the longest run of a wave set the time, took 256 us for
// 28,000 queries; this takes 45, the workgroups' kernel after it 13.)
template <int K>
__global__ __launch_bounds__(256) void k_dc_knn_wave(int n, const float4* __restrict__ pts,
                                                     const uint32_t* __restrict__ start, uint32_t T, float h, float inv_h,
                                                     const uint32_t* __restrict__ far, const uint32_t* __restrict__ far_n,
                                                     uint32_t* __restrict__ far2, uint32_t* __restrict__ far2_n,
                                                     int32_t* __restrict__ nn, float* __restrict__ dnn,
                                                     float* __restrict__ dbar, DcSums* __restrict__ sums) {
  __shared__ uint32_t s_end[8][64], s_at[8][64];   // 7^2 runs, to whole rounds of the lanes
  const int half = threadIdx.x >> 5;
  const uint32_t count = *far_n;
  double a1 = 0.0, a2 = 0.0;
  for (uint32_t f = blockIdx.x * 8 + half; f < count; f += gridDim.x * 8) {
    const uint32_t slot = far[f];
    const float4 q = pts[slot];
    double b[K];
    const bool done =
        n - 1 >= K && (dc_search<K, 2, 32>(b, n, pts, start, T, h, inv_h, q, s_end[half], s_at[half], nullptr) ||
                       dc_search<K, 3, 32>(b, n, pts, start, T, h, inv_h, q, s_end[half], s_at[half], nullptr));
    if ((threadIdx.x & 31) == 0) {
      if (done) {
        const double d0 = static_cast<double>(dc_finish<K>(b, K, __float_as_int(q.w), nn, dnn, dbar));
        a1 += d0;
        a2 += d0 * d0;
      } else {
        far2[atomicAdd(far2_n, 1u)] = slot;
      }
    }
  }
  if ((threadIdx.x & 31) == 0 && a2 != 0.0) {
    DcSums* d = sums + (blockIdx.x * 8 + half) % kDcSlots;
    unsafeAtomicAdd(&d->a1, a1);
    unsafeAtomicAdd(&d->a2, a2);
  }
}

// Queries still open, a workgroup each: the cells up to R = 7.  (Half a wave took
// some 20 us for one of these, and they come in clusters, so that the last of the
// kernel before doubled its time.)  What is left goes to the scan of every point.
template <int K>
__global__ __launch_bounds__(256) void k_dc_knn_wide(int n, const float4* __restrict__ pts,
                                                     const uint32_t* __restrict__ start, uint32_t T, float h, float inv_h,
                                                     const uint32_t* __restrict__ far, const uint32_t* __restrict__ far_n,
                                                     uint32_t* __restrict__ far2, uint32_t* __restrict__ far2_n,
                                                     int32_t* __restrict__ nn, float* __restrict__ dnn,
                                                     float* __restrict__ dbar, DcSums* __restrict__ sums) {
  __shared__ uint32_t s_end[256], s_at[256];   // 15^2 runs
  __shared__ double s_lists[4 * K];
  const uint32_t count = *far_n;
  for (uint32_t f = blockIdx.x; f < count; f += gridDim.x) {
    const uint32_t slot = far[f];
    const float4 q = pts[slot];
    double b[K];
    const bool done = n - 1 >= K && dc_search<K, 7, 256>(b, n, pts, start, T, h, inv_h, q, s_end, s_at, s_lists);
    if (threadIdx.x == 0) {
      if (done) {
        const double d0 = static_cast<double>(dc_finish<K>(b, K, __float_as_int(q.w), nn, dnn, dbar));
        unsafeAtomicAdd(&sums[blockIdx.x % kDcSlots].a1, d0);
        unsafeAtomicAdd(&sums[blockIdx.x % kDcSlots].a2, d0 * d0);
      } else {
        far2[atomicAdd(far2_n, 1u)] = slot;
      }
    }
  }
}

// The queries the searches left (fewer than K other points: every query): a
// workgroup per (query, range of points) scans its range (each thread a strided
// share, its own K best) and merges the 256 lists; with S > 1 ranges the lists
// go to cand for k_dc_knn_far_merge, with one range the result is written here.
// Splitting keeps a few isolated queries from each holding one workgroup
// over every point (at 1M Gaussians, 44 queries took 1.7 ms that way).
template <int K>
__global__ __launch_bounds__(256) void k_dc_knn_far(int n, const float4* __restrict__ pts,
                                                    const uint32_t* __restrict__ far, const uint32_t* __restrict__ far_n,
                                                    int32_t* __restrict__ nn, float* __restrict__ dnn,
                                                    float* __restrict__ dbar, DcSums* __restrict__ sums,
                                                    double* __restrict__ cand) {
  __shared__ double s_b[4][K];
  const uint32_t count = *far_n;
  const uint32_t S = far_splits(count);
  const uint32_t span = (static_cast<uint32_t>(n) + S - 1u) / S;
  // items (query f, range r): points [r span, (r + 1) span)
  for (uint32_t it = blockIdx.x; it < count * S; it += gridDim.x) {
    const uint32_t f = it / S, r = it - f * S;
    const float4 q = pts[far[f]];
    const int qi = __float_as_int(q.w);
    double b[K];
#pragma unroll
    for (int m = 0; m < K; ++m) b[m] = dc_empty();
    const int p0 = static_cast<int>(r * span), p1 = min(n, static_cast<int>((r + 1u) * span));
    for (int p = p0 + threadIdx.x; p < p1; p += 256) {
      const float4 o = pts[p];
      const int oi = __float_as_int(o.w);
      dc_insert<K>(b, dc_key(oi != qi ? dc_d2(q, o) : dc_none(), oi));
    }
    dc_merge64<K>(b);
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
      for (int m = 0; m < K; ++m) s_b[threadIdx.x >> 6][m] = b[m];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int w = 1; w < 4; ++w)
        for (int m = 0; m < K; ++m) dc_insert<K>(b, s_b[w][m]);
      if (S == 1) {
        const double d0 = static_cast<double>(dc_finish<K>(b, min(K, n - 1), qi, nn, dnn, dbar));
        unsafeAtomicAdd(&sums[blockIdx.x % kDcSlots].a1, d0);
        unsafeAtomicAdd(&sums[blockIdx.x % kDcSlots].a2, d0 * d0);
      } else {
#pragma unroll
        for (int m = 0; m < K; ++m) cand[static_cast<size_t>(it) * 8 + m] = b[m];
      }
    }
    __syncthreads();
  }
}

// Merge of the split far search: query f's K nearest among its S ranges'
// lists, in (distance, index) order as every search keeps them.  One wave per
// query: lane r takes range r's list (r < S <= 64), and the lists are merged
// over the wave (exact: the order is total).
template <int K>
__global__ __launch_bounds__(64) void k_dc_knn_far_merge(int n, const float4* __restrict__ pts,
                                                         const uint32_t* __restrict__ far,
                                                         const uint32_t* __restrict__ far_n, int32_t* __restrict__ nn,
                                                         float* __restrict__ dnn, float* __restrict__ dbar,
                                                         DcSums* __restrict__ sums, const double* __restrict__ cand) {
  const uint32_t count = *far_n;
  const uint32_t S = far_splits(count);
  if (S == 1u) return;
  const uint32_t lane = threadIdx.x;
  for (uint32_t f = blockIdx.x; f < count; f += gridDim.x) {
    double b[K];
#pragma unroll
    for (int m = 0; m < K; ++m) b[m] = lane < S ? cand[(static_cast<size_t>(f) * S + lane) * 8 + m] : dc_empty();
    dc_merge64<K>(b);
    if (lane == 0) {
      const int qi = __float_as_int(pts[far[f]].w);
      const double d0 = static_cast<double>(dc_finish<K>(b, min(K, n - 1), qi, nn, dnn, dbar));
      unsafeAtomicAdd(&sums[f % kDcSlots].a1, d0);
      unsafeAtomicAdd(&sums[f % kDcSlots].a2, d0 * d0);
    }
  }
}

// The thresholds from the statistics' sums (every wave adds the slots up by
// itself, in the same order): mu = S1/n, sigma = sqrt(max(S2/n - mu^2, 0)),
// rho_low = mu - alpha sigma, rho_high = mu + beta sigma from the exact integer
// sums in FP64 with correctly rounded operations, and d_merge = mu_d + gamma
// sigma_d over the nearest distances; then each point's class and the merge
// pairing: pos[i] = 0 for the higher index of a merged pair, pos[n + i] = 1 for
// a point that spawns a new one.
__global__ __launch_bounds__(256) void k_dc_classify(int n, const int32_t* __restrict__ rho,
                                                     const int32_t* __restrict__ nn, const float* __restrict__ dnn,
                                                     const DcSums* __restrict__ sums, double alpha, double beta,
                                                     double gamma, DcReport* __restrict__ rep,
                                                     uint32_t* __restrict__ pos, int32_t* __restrict__ partner,
                                                     uint8_t* __restrict__ cls_out) {
  const DcSums mine = sums[threadIdx.x & (kDcSlots - 1u)];
  unsigned long long c1 = mine.c1, c2 = mine.c2;
  double a1 = mine.a1, a2 = mine.a2;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    c1 += __shfl_xor(c1, o, 64);
    c2 += __shfl_xor(c2, o, 64);
    a1 += __shfl_xor(a1, o, 64);
    a2 += __shfl_xor(a2, o, 64);
  }
  const double dn = static_cast<double>(n);
  const double mu = __ddiv_rn(static_cast<double>(c1), dn);
  const double var = __dsub_rn(__ddiv_rn(static_cast<double>(c2), dn), __dmul_rn(mu, mu));
  const double sigma = __dsqrt_rn(var > 0.0 ? var : 0.0);
  const double lo = __dsub_rn(mu, __dmul_rn(alpha, sigma)), hi = __dadd_rn(mu, __dmul_rn(beta, sigma));
  const double mud = n > 1 ? a1 / dn : 0.0;
  const double vard = n > 1 ? a2 / dn - mud * mud : 0.0;
  const double sigmad = sqrt(vard > 0.0 ? vard : 0.0);
  const double dm = mud + gamma * sigmad;
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i == 0) {
    rep->stat[0] = mu; rep->stat[1] = sigma; rep->stat[2] = lo; rep->stat[3] = hi;
    rep->stat[4] = mud; rep->stat[5] = sigmad; rep->stat[6] = dm;
  }
  if (i >= n) return;
  auto cls = [&](int k) -> int {
    const double r = static_cast<double>(rho[k]);
    return r < lo ? 1 : (r > hi ? 2 : 0);
  };
  const int c = cls(i);
  const int j = nn[i];
  const bool pair = c == 2 && j >= 0 && j < n && cls(j) == 2 && nn[j] == i && static_cast<double>(dnn[i]) <= dm;
  partner[i] = pair ? j : -1;
  pos[i] = (pair && j < i) ? 0u : 1u;
  pos[static_cast<int64_t>(n) + i] = c == 1 ? 1u : 0u;
  if (cls_out) cls_out[i] = static_cast<uint8_t>(c);
}

__device__ __forceinline__ float dc_sigmoid(float x) { return 1.0f / (1.0f + expf(-x)); }
__device__ __forceinline__ float dc_softplus(float x) { return x > 0.0f ? x + log1pf(expf(-x)) : log1pf(expf(x)); }

struct DcArrays {
  const float *means, *ls, *quats, *logits, *sh;
  float *o_means, *o_ls, *o_quats, *o_logits, *o_sh;
  int64_t cap;
  int nsh;  // 3 (D + 1)^2
};

constexpr int kDcComps = 12;   // spherical-harmonics planes that a workgroup of k_dc_write copies

// Output of every point: its own values, a merged pair's (at the lower index),
// and a new point next to each sparse point (after all kept points).  Workgroup
// row 0 writes the geometry, row y > 0 the colour planes 12 (y - 1) to 12 y - 1.
// HBM bounds it: 190 MB past the L2s (kept points move to where the cache lines no
// longer match) in 40 us at 200,000 points, 4.8 TB/s; one thread per point, all planes
// in turn, took 61.
__global__ __launch_bounds__(256) void k_dc_write(int n, DcArrays A, const uint32_t* __restrict__ pos,
                                                  const int32_t* __restrict__ partner, const float* __restrict__ dbar,
                                                  const float* __restrict__ noise, float spread, float jitter,
                                                  DcReport* __restrict__ rep, int32_t* __restrict__ fate) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int64_t N = n, cap = A.cap;
  const int j = partner[i];
  const bool kept = !(j >= 0 && j < i);
  const int64_t o = static_cast<int64_t>(pos[i]);
  // where a new point goes; the flag itself is recovered from the next prefix (or the total)
  const int64_t q = static_cast<int64_t>(pos[N + i]);
  const int64_t next = i + 1 < n ? static_cast<int64_t>(pos[N + i + 1]) : static_cast<int64_t>(rep->total);
  const bool put = kept && o < cap, spawn = next > q && q < cap;
  const bool merged = put && j >= 0;
  float oi = 1.0f, oj = 0.0f, li = 0.0f, lj = 0.0f;
  if (merged) {
    li = A.logits[i]; lj = A.logits[j];
    oi = dc_sigmoid(li); oj = dc_sigmoid(lj);
  }
  const float w = oi + oj;
  if (blockIdx.y > 0) {
    const int c0 = (static_cast<int>(blockIdx.y) - 1) * kDcComps, c1 = min(c0 + kDcComps, A.nsh);
    if (!(put || spawn)) return;
    // all loads first, so that they are in flight together
    float v[kDcComps], u[kDcComps];
#pragma unroll
    for (int c = 0; c < kDcComps; ++c) v[c] = c0 + c < c1 ? __builtin_nontemporal_load(&A.sh[(c0 + c) * N + i]) : 0.0f;
    if (merged) {
#pragma unroll
      for (int c = 0; c < kDcComps; ++c) u[c] = c0 + c < c1 ? A.sh[(c0 + c) * N + j] : 0.0f;
    }
    if (spawn) {
#pragma unroll
      for (int c = 0; c < kDcComps; ++c)
        if (c0 + c < c1) __builtin_nontemporal_store(v[c], &A.o_sh[(c0 + c) * cap + q]);
    }
    if (merged) {
#pragma unroll
      for (int c = 0; c < kDcComps; ++c) v[c] = (oi * v[c] + oj * u[c]) / w;
    }
    if (put) {
#pragma unroll
      for (int c = 0; c < kDcComps; ++c)
        if (c0 + c < c1) __builtin_nontemporal_store(v[c], &A.o_sh[(c0 + c) * cap + o]);
    }
    return;
  }
  if (i == 0) rep->kept = pos[N];
  if (fate) fate[i] = kept ? static_cast<int32_t>(o) : -1;
  if (put) {
    if (j < 0) {
      for (int c = 0; c < 3; ++c) {
        A.o_means[c * cap + o] = A.means[c * N + i];
        A.o_ls[c * cap + o] = A.ls[c * N + i];
      }
      for (int c = 0; c < 4; ++c) A.o_quats[c * cap + o] = A.quats[c * N + i];
      A.o_logits[o] = A.logits[i];
    } else {
      // merge with j (j > i): opacity-weighted position and colour, mean
      // scale, accumulated opacity, the more opaque one's rotation
      for (int c = 0; c < 3; ++c) {
        A.o_means[c * cap + o] = (oi * A.means[c * N + i] + oj * A.means[c * N + j]) / w;
        A.o_ls[c * cap + o] = logf(0.5f * (expf(A.ls[c * N + i]) + expf(A.ls[c * N + j])));
      }
      const int qs = oj > oi ? j : i;
      for (int c = 0; c < 4; ++c) A.o_quats[c * cap + o] = A.quats[c * N + qs];
      // logit of 1 - (1 - oi)(1 - oj): log(o) + softplus(li) + softplus(lj)
      A.o_logits[o] = logf(oi + oj - oi * oj) + dc_softplus(li) + dc_softplus(lj);
    }
  }
  if (spawn) {
    const float t = __fmul_rn(spread, dbar[i]);
    for (int c = 0; c < 3; ++c) {
      float p = __fadd_rn(A.means[c * N + i], __fmul_rn(t, noise[c * N + i]));
      p = __fadd_rn(p, __fmul_rn(jitter, noise[(3 + c) * N + i]));
      A.o_means[c * cap + q] = p;
      A.o_ls[c * cap + q] = A.ls[c * N + i];
    }
    for (int c = 0; c < 4; ++c) A.o_quats[c * cap + q] = A.quats[c * N + i];
    A.o_logits[q] = A.logits[i];
  }
}

gs_status launch_density_control(const gs_gaussians& g, const gs_density_params& prm, const float* noise,
                                 gs_param_arrays& out, int64_t cap, void* ws, gs_density_report* rep,
                                 gs_density_points* pts_out, hipStream_t s) {
  const int n = static_cast<int>(g.n);
  DcWs w = carve_dc(ws, n);
  const uint32_t T = dc_table(n);
  const float h = prm.radius * kDcCellScale;
  const float inv_h = 1.0f / h;
  const float r2 = prm.radius * prm.radius;  // r r, rounded once
  const unsigned gn = static_cast<unsigned>(std::max<int64_t>(ceil_div(n, 256), 1));
  gs_status st;
  DcReport r{};
  if (n > 0) {
    { TimedLaunch t("k_dc_clear", s); k_dc_clear<<<static_cast<unsigned>(ceil_div(T, 256)), 256, 0, s>>>(w.count, T, w.sums, w.rep,
                                                                                                 w.far_n, w.far2_n, w.far3_n); }
    if ((st = check_launch("k_dc_clear")) != GS_OK) return st;
    { TimedLaunch t("k_dc_cells", s); k_dc_cells<<<gn, 256, 0, s>>>(n, g.means, inv_h, T - 1u, w.cell, w.count, w.rep); }
    if ((st = check_launch("k_dc_cells")) != GS_OK) return st;
    if ((st = launch_exclusive_scan(w.count, w.count, T, w.scan, nullptr, s)) != GS_OK) return st;
    { TimedLaunch t("k_dc_scatter", s); k_dc_scatter<<<gn, 256, 0, s>>>(n, g.means, w.cell, w.count, w.pts); }
    if ((st = check_launch("k_dc_scatter")) != GS_OK) return st;
#define GS_DC_KNN(K)                                                                                              \
  {                                                                                                               \
    { TimedLaunch t("k_dc_near<" #K ">", s);                                                                      \
      k_dc_near<K><<<static_cast<unsigned>(ceil_div(n, 256 / kDcLanes)), 256, 0, s>>>(n, w.pts, w.count, T, h, inv_h, r2, w.rho, \
                                                                          w.nn, w.dnn, w.dbar, w.sums, w.far,     \
                                                                          w.far_n); }                             \
    { TimedLaunch t("k_dc_knn_wave<" #K ">", s);                                                                  \
      k_dc_knn_wave<K><<<2048, 256, 0, s>>>(n, w.pts, w.count, T, h, inv_h, w.far, w.far_n, w.far2, w.far2_n,     \
                                            w.nn, w.dnn, w.dbar, w.sums); }                                       \
    { TimedLaunch t("k_dc_knn_wide<" #K ">", s);                                                                  \
      k_dc_knn_wide<K><<<1024, 256, 0, s>>>(n, w.pts, w.count, T, h, inv_h, w.far2, w.far2_n, w.far, w.far3_n,    \
                                            w.nn, w.dnn, w.dbar, w.sums); }                                       \
    { TimedLaunch t("k_dc_knn_far<" #K ">", s);                                                                   \
      k_dc_knn_far<K><<<1024, 256, 0, s>>>(n, w.pts, w.far, w.far3_n, w.nn, w.dnn, w.dbar, w.sums, w.cand); }     \
    { TimedLaunch t("k_dc_knn_far_merge<" #K ">", s);                                                             \
      k_dc_knn_far_merge<K><<<256, 64, 0, s>>>(n, w.pts, w.far, w.far3_n, w.nn, w.dnn, w.dbar, w.sums, w.cand); } \
  }
    switch (prm.knn) {
      case 1: GS_DC_KNN(1); break;
      case 2: GS_DC_KNN(2); break;
      case 3: GS_DC_KNN(3); break;
      case 4: GS_DC_KNN(4); break;
      case 5: GS_DC_KNN(5); break;
      case 6: GS_DC_KNN(6); break;
      case 7: GS_DC_KNN(7); break;
      default: GS_DC_KNN(8); break;
    }
#undef GS_DC_KNN
    if ((st = check_launch("k_dc_knn")) != GS_OK) return st;
    { TimedLaunch t("k_dc_classify", s);
      k_dc_classify<<<gn, 256, 0, s>>>(n, w.rho, w.nn, w.dnn, w.sums, static_cast<double>(prm.alpha),
                                       static_cast<double>(prm.beta), static_cast<double>(prm.gamma), w.rep, w.pos,
                                       w.partner, pts_out ? pts_out->cls : nullptr); }
    if ((st = check_launch("k_dc_classify")) != GS_OK) return st;
    if (pts_out) {
      if (pts_out->rho && (st = check_hip(hipMemcpyAsync(pts_out->rho, w.rho, sizeof(int32_t) * n, hipMemcpyDeviceToDevice, s),
                                          "hipMemcpyAsync(rho)")) != GS_OK) return st;
      if (pts_out->nn && (st = check_hip(hipMemcpyAsync(pts_out->nn, w.nn, sizeof(int32_t) * n, hipMemcpyDeviceToDevice, s),
                                         "hipMemcpyAsync(nn)")) != GS_OK) return st;
      if (pts_out->dbar && (st = check_hip(hipMemcpyAsync(pts_out->dbar, w.dbar, sizeof(float) * n, hipMemcpyDeviceToDevice, s),
                                           "hipMemcpyAsync(dbar)")) != GS_OK) return st;
    }
    if ((st = launch_exclusive_scan(w.pos, w.pos, 2 * static_cast<int64_t>(n), w.scan, &w.rep->total, s)) != GS_OK) return st;
    DcArrays A{g.means, g.log_scales, g.quats, g.logits, g.sh,
               out.means, out.log_scales, out.quats, out.logits, out.sh, cap, 3 * (g.sh_degree + 1) * (g.sh_degree + 1)};
    const dim3 gw(gn, 1u + static_cast<unsigned>(ceil_div(A.nsh, kDcComps)));
    { TimedLaunch t("k_dc_write", s); k_dc_write<<<gw, 256, 0, s>>>(n, A, w.pos, w.partner, w.dbar, noise, prm.spread, prm.jitter,
                                                                 w.rep, pts_out ? pts_out->fate : nullptr); }
    if ((st = check_launch("k_dc_write")) != GS_OK) return st;
    if ((st = check_hip(hipMemcpyAsync(&r, w.rep, sizeof r, hipMemcpyDeviceToHost, s), "hipMemcpyAsync(report)")) != GS_OK)
      return st;
    if ((st = check_hip(hipStreamSynchronize(s), "hipStreamSynchronize")) != GS_OK) return st;
    if (r.range)
      return fail(GS_ERR_UNSUPPORTED, "gs_density_control: a coordinate is not finite or lies 2^18 cells (of 1.07 r) "
                                      "or more from the origin; the outputs are undefined");
    if (rep) {
      rep->rho_mean = r.stat[0]; rep->rho_std = r.stat[1]; rep->rho_low = r.stat[2]; rep->rho_high = r.stat[3];
      rep->d_mean = r.stat[4]; rep->d_std = r.stat[5]; rep->d_merge = r.stat[6];
    }
  }
  const int64_t kept = static_cast<int64_t>(r.kept), total = static_cast<int64_t>(r.total);
  if (rep) {
    rep->n_in = n;
    rep->n_merged = n - kept;
    rep->n_new = total - kept;
    rep->n_out = total;
  }
  if (total > cap)
    return fail(GS_ERR_CAPACITY, "gs_density_control: the output needs " + std::to_string(total) +
                                     " Gaussians, the capacity is " + std::to_string(cap));
  return GS_OK;
}

}  // namespace gs
