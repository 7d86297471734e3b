// Learned colour decoder on the BF16 matrix cores (v_mfma_f32_16x16x32_bf16).
//
// Not part of the paper's method: an optional replacement for the SH colour
// read of the projection (Sec. I / Sec. II-A, colour from SH coefficients).
// Per sample, x = [z (16 latent values); Y_0..15(d)] (the real SH encoding of
// the unit view direction), h1 = ReLU(W1 x + b1), h2 = ReLU(W2 h1 + b2),
// c = sigmoid(W3 h2 + b3); W and z are BF16, every product is accumulated in
// FP32, and the view encoding and hidden activations enter the products as a
// hi + lo pair of BF16 values (about 2^-17 relative), so the colour matches the
// BF16-weight definition to near FP32 accuracy.
//
// A wave evaluates 16 samples at a time.  In the 16x16x32 MFMA, lane l holds
// A[l % 16][8 (l / 16) + e], B[8 (l / 16) + e][l % 16] (e = 0..7) and
// D[4 (l / 16) + i][l % 16] (i = 0..3).  Samples run along the 16 columns, so
// after a layer lane l holds hidden units 16 b + 4 (l / 16) + i of sample
// l % 16.  Read back as the next layer's B operand, slot e of lane l then
// carries hidden unit hid(c, l / 16, e) = 32 c + 16 (e / 4) + 4 (l / 16) + e % 4
// of k-chunk c; the packed weights permute their input columns the same way,
// so activations never leave registers between layers.
#include "gs_internal.h"
#include "gs_sh.h"

namespace gs {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kMlpIn = 32, kMlpH = 64, kMlpOut = 3;
constexpr int P_W1 = 0, P_B1 = 2048, P_W2 = 2112, P_B2 = 6208, P_W3 = 6272, P_B3 = 6464;

// Packed operand image: kOps tiles of 64 lanes x 8 BF16 values, then the
// biases in FP32 (b1[64], b2[64], b3[3]).
//   0..3   W1 row-block b                       (forward, layer 1)
//   4..11  W2 row-block b, k-chunk c (4+2b+c)    (forward, layer 2, permuted k)
//   12..13 W3 (rows 3..15 zero), k-chunk c       (forward, layer 3, permuted k)
//   14..17 W3^T row-block b (k = output unit)    (backward, dL/dh2)
//   18..25 W2^T row-block b, k-chunk c (18+2b+c) (backward, dL/dh1, permuted k)
//   26..29 W1^T row-block b, k-chunk c (26+2b+c) (backward, dL/dx, permuted k)
constexpr int kOps = 30;
constexpr int kOpW1 = 0, kOpW2 = 4, kOpW3 = 12, kOpW3T = 14, kOpW2T = 18, kOpW1T = 26;
constexpr int kBiasFloats = 131;

__host__ __device__ constexpr int hid(int c, int g, int e) { return 32 * c + 16 * (e >> 2) + 4 * g + (e & 3); }

__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float(static_cast<uint32_t>(b) << 16); }

__device__ __forceinline__ floatx4 mfma(const uint4& a, const bf16x8& b, const floatx4& c) {
  bf16x8 av;
  __builtin_memcpy(&av, &a, sizeof(av));
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, b, c, 0, 0, 0);
}

__global__ __launch_bounds__(64) void k_mlp_pack(const uint16_t* __restrict__ P, uint4* __restrict__ ops,
                                                 float* __restrict__ bias) {
  const int op = blockIdx.x, l = threadIdx.x, g = l >> 4, r = l & 15;
  uint16_t v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    uint16_t x = 0;
    if (op < kOpW2) {
      x = P[P_W1 + (16 * op + r) * kMlpIn + 8 * g + e];
    } else if (op < kOpW3) {
      const int b = (op - kOpW2) >> 1, c = (op - kOpW2) & 1;
      x = P[P_W2 + (16 * b + r) * kMlpH + hid(c, g, e)];
    } else if (op < kOpW3T) {
      const int c = op - kOpW3;
      x = (r < kMlpOut) ? P[P_W3 + r * kMlpH + hid(c, g, e)] : 0;
    } else if (op < kOpW2T) {
      const int b = op - kOpW3T;
      x = (g == 0 && e < kMlpOut) ? P[P_W3 + e * kMlpH + 16 * b + r] : 0;
    } else if (op < kOpW1T) {
      const int b = (op - kOpW2T) >> 1, c = (op - kOpW2T) & 1;
      x = P[P_W2 + hid(c, g, e) * kMlpH + 16 * b + r];
    } else {
      const int b = (op - kOpW1T) >> 1, c = (op - kOpW1T) & 1;
      x = P[P_W1 + hid(c, g, e) * kMlpIn + 16 * b + r];
    }
    v[e] = x;
  }
  uint4 w;
  w.x = v[0] | (static_cast<uint32_t>(v[1]) << 16);
  w.y = v[2] | (static_cast<uint32_t>(v[3]) << 16);
  w.z = v[4] | (static_cast<uint32_t>(v[5]) << 16);
  w.w = v[6] | (static_cast<uint32_t>(v[7]) << 16);
  ops[op * 64 + l] = w;
  if (op == 0) {
    bias[l] = bf2f(P[P_B1 + l]);
    bias[64 + l] = bf2f(P[P_B2 + l]);
    if (l < kMlpOut) bias[128 + l] = bf2f(P[P_B3 + l]);
  }
}

struct MlpShared {
  uint4 ops[kOps * 64];
  float bias[kBiasFloats + 1];
};

__device__ __forceinline__ void load_packed(MlpShared& sh, const uint4* __restrict__ ops,
                                            const float* __restrict__ bias) {
  for (int i = threadIdx.x; i < kOps * 64; i += blockDim.x) sh.ops[i] = ops[i];
  for (int i = threadIdx.x; i < kBiasFloats; i += blockDim.x) sh.bias[i] = bias[i];
}

// A value v carried as two BF16 operands, hi = bf16(v) and lo = bf16(v - hi):
// hi + lo equals v to about 2^-17 relative, so products with the (exactly
// BF16) weights keep activations and the view encoding at close to FP32
// accuracy for twice the matrix-core work, which is not this kernel's bound.
struct Split8 {
  bf16x8 hi, lo;
};

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

// Two values split at once: one packed conversion for both hi parts, one for
// both lo parts (round to nearest even, as a single conversion would).
struct Split2 {
  bf16x2 hi, lo;
};
__device__ __forceinline__ Split2 split2(float a, float b) {
  const floatx2 v = {a, b};
  Split2 p;
  p.hi = __builtin_convertvector(v, bf16x2);
  p.lo = __builtin_convertvector(v - __builtin_convertvector(p.hi, floatx2), bf16x2);
  return p;
}

// slots e, e + 1 (e even) of s
__device__ __forceinline__ void split_put2(Split8& s, int e, float a, float b) {
  const Split2 p = split2(a, b);
  s.hi[e] = p.hi[0]; s.hi[e + 1] = p.hi[1];
  s.lo[e] = p.lo[0]; s.lo[e + 1] = p.lo[1];
}

// D-layout values (4 row-blocks) as the split B operands of the next product.
__device__ __forceinline__ void d_to_b(const floatx4 h[4], Split8& B0, Split8& B1) {
#pragma unroll
  for (int e = 0; e < 8; e += 2) {
    split_put2(B0, e, h[e >> 2][e & 3], h[e >> 2][(e & 3) + 1]);
    split_put2(B1, e, h[2 + (e >> 2)][e & 3], h[2 + (e >> 2)][(e & 3) + 1]);
  }
}

// Where a layer's pre-activations are positive, a wave mask per value (scalar
// registers: the backward needs them long after the values).
struct ReluMask {
  uint64_t m[4][4];
};

// The split ReLU of a layer's pre-activations (0 for a NaN) and their signs.
__device__ __forceinline__ void relu_to_b(const floatx4 h[4], Split8& B0, Split8& B1, ReluMask& on) {
  floatx4 p[4];
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      on.m[b][i] = __builtin_amdgcn_ballot_w64(h[b][i] > 0.0f);
      p[b][i] = __builtin_amdgcn_inverse_ballot_w64(on.m[b][i]) ? h[b][i] : 0.0f;
    }
  d_to_b(p, B0, B1);
}

// The biases of a hidden layer in the D layout of row-block b: lane (g, r)
// holds rows 4 g .. 4 g + 3, i.e. units 16 b + 4 g + i -- the accumulator a
// layer's products start from, so the pre-activation needs no separate add.
__device__ __forceinline__ floatx4 bias_d(const float* bias, int b, int g) {
  return *reinterpret_cast<const floatx4*>(bias + 16 * b + 4 * g);
}

// Layer-1 B operand of lane (g, sample s): latent values 8g..8g+7 (g < 2,
// exact BF16, lo = 0) or the SH encoding values 8(g-2)..8(g-2)+7 of the view
// direction (g >= 2).
__device__ __forceinline__ Split8 input_operand(int g, bool valid, const uint4& zslice, const float d[3]) {
  Split8 X;
  if (g < 2) {
    const uint4 raw = valid ? zslice : make_uint4(0, 0, 0, 0);
    __builtin_memcpy(&X.hi, &raw, sizeof(X.hi));
#pragma unroll
    for (int e = 0; e < 8; ++e) X.lo[e] = static_cast<__bf16>(0.0f);
  } else {
    float Y[16];
    sh_basis(3, d[0], d[1], d[2], Y);
    // static indices (a lane-dependent index into Y would become a select chain)
    const bool upper = g == 3;
#pragma unroll
    for (int e = 0; e < 8; e += 2)
      split_put2(X, e, valid ? (upper ? Y[8 + e] : Y[e]) : 0.0f, valid ? (upper ? Y[9 + e] : Y[e + 1]) : 0.0f);
  }
  return X;
}

// N consecutive packed tiles, read together (one wait for all).
template <int N>
__device__ __forceinline__ void tiles(const MlpShared& sh, int op, int lane, uint4* w) {
#pragma unroll
  for (int k = 0; k < N; ++k) w[k] = sh.ops[(op + k) * 64 + lane];
}

// Staging of one group ([sample][unit]); plane 0 holds the BF16 value (hi),
// plane 1 the BF16 rounding of the remainder (lo).  Rows of 64 units are padded
// to 72 (36 banks): the stores of a quarter's 16 lanes (one per row) and the
// transposing reads (32 bytes of four rows) then each touch different banks.
constexpr int kRow = 72, kRowX = 36, kRowG3 = 4;
struct alignas(16) MlpStage {
  __bf16 h1[2][16][kRow];
  __bf16 g1[2][16][kRow];
  __bf16 hg2[2][16][kRow];   // h2, then g2
  __bf16 x[2][16][kRowX];
  __bf16 g3[2][16][kRowG3];
};

typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// Orders a wave's LDS accesses: its lanes read what other lanes of it wrote.
// (The hardware keeps a wave's LDS operations in order; this keeps the compiler.)
__device__ __forceinline__ void stage_fence() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// The split operands of k-chunks 0, 1 of sample r: slots 4 q .. 4 q + 3 of chunk c
// are units 32 c + 16 q + 4 g and the three after it.
__device__ __forceinline__ void stage_put(__bf16 (*m)[16][kRow], int g, int r, const Split8& S0, const Split8& S1) {
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const Split8& S = c ? S1 : S0;
      const int at = 32 * c + 16 * q + 4 * g;
      const bf16x4 hi = {S.hi[4 * q], S.hi[4 * q + 1], S.hi[4 * q + 2], S.hi[4 * q + 3]};
      const bf16x4 lo = {S.lo[4 * q], S.lo[4 * q + 1], S.lo[4 * q + 2], S.lo[4 * q + 3]};
      __builtin_memcpy(&m[0][r][at], &hi, sizeof(hi));
      __builtin_memcpy(&m[1][r][at], &lo, sizeof(lo));
    }
}

// Samples 4 g .. 4 g + 3 of unit 16 b + r of a staged plane.  The transposing read
// works on 16 lanes: lane r names row r / 4 (of four), columns 4 (r % 4) .. + 3 (of
// sixteen), and gets column r of the four rows.  (g3 has four columns: its rows
// come back four times.)
template <int ROW>
__device__ __forceinline__ bf16x4 stage_get(const __bf16 (*p)[ROW], int b, int g, int r) {
  auto* at = reinterpret_cast<const __attribute__((address_space(3))) shortx4*>(
      reinterpret_cast<uintptr_t>(&p[4 * g + (r >> 2)][ROW > 4 ? 16 * b + 4 * (r & 3) : 0]));
  const shortx4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(const_cast<__attribute__((address_space(3))) shortx4*>(at));
  bf16x4 o;
  __builtin_memcpy(&o, &v, sizeof(o));
  return o;
}

__device__ __forceinline__ bf16x8 join(const bf16x4& a, const bf16x4& b) {
  return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}

struct MlpFwdState {
  floatx4 o;
  Split8 X, B0, B1, C0, C1;
  ReluMask m1, m2;
};

__device__ __forceinline__ floatx4 mfma2(const uint4& a, const Split8& b, const floatx4& c) {
  return mfma(a, b.lo, mfma(a, b.hi, c));
}

// B, C: the split ReLU outputs; m1, m2: the signs of the pre-activations.  BWD:
// the activations also go to sg, as soon as they are there.
template <bool BWD>
__device__ __forceinline__ void mlp_forward_group(const MlpShared& sh, int lane, MlpFwdState& st, MlpStage* sg = nullptr) {
  const int g = lane >> 4;
  const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
  floatx4 h[4];
  uint4 w[8];
  tiles<4>(sh, kOpW1, lane, w);
#pragma unroll
  for (int b = 0; b < 4; ++b) h[b] = mfma2(w[b], st.X, bias_d(sh.bias, b, g));
  tiles<8>(sh, kOpW2, lane, w);
  relu_to_b(h, st.B0, st.B1, st.m1);
  if (BWD) stage_put(sg->h1, g, lane & 15, st.B0, st.B1);
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const floatx4 acc = mfma2(w[2 * b], st.B0, bias_d(sh.bias + 64, b, g));
    h[b] = mfma2(w[2 * b + 1], st.B1, acc);
  }
  tiles<2>(sh, kOpW3, lane, w);
  relu_to_b(h, st.C0, st.C1, st.m2);
  if (BWD) stage_put(sg->hg2, g, lane & 15, st.C0, st.C1);
  st.o = mfma2(w[1], st.C1, mfma2(w[0], st.C0, zero));
}

// The hardware reciprocal (1 ulp) instead of a correctly rounded division:
// the colour's error budget is set by the BF16 products, far above it.
__device__ __forceinline__ float sigmoidf(float x) { return __builtin_amdgcn_rcpf(1.0f + __expf(-x)); }

// Inputs of one lane's sample.  The kernels load them one group ahead, so
// their latency hides behind the current group's arithmetic (a wave runs
// many groups in turn and few waves share a SIMD).
struct SampleIn {
  float a[3];       // unit direction (MODE 0) or the Gaussian's mean (MODE 1)
  float c[3];       // backward: dL/dc or the distillation target (quarter 0)
  uint4 z;          // latent values 8 g .. 8 g + 7 (quarters 0, 1)
  float m[3];       // MODE 1 backward: dL/dmean so far (the geometry's share)
  bool in;          // s < S (and, MODE 1, the Gaussian is live)
};

// dL_dc: channel i of sample s at dL_dc[(c0 + i) cs + s ss] -- MODE 0 [S][3]
// (c0 0, cs 1, ss 3); MODE 1 g2d[9][S] (c0 6, cs S, ss 1) or accumulator rows
// [S][kAccStride] (c0 6, cs 1, ss kAccStride).
template <int MODE, bool BWD>
__device__ __forceinline__ SampleIn load_sample(int64_t s64, int S, int per, int g, const uint16_t* __restrict__ latents,
                                                const float* __restrict__ dirs, const float* __restrict__ means,
                                                const int* __restrict__ radius, const float* __restrict__ dL_dc,
                                                const float* __restrict__ dmean = nullptr, int64_t cs = 1,
                                                int64_t ss = 3) {
  SampleIn x;
  x.a[0] = 0.f; x.a[1] = 0.f; x.a[2] = 1.f;
  x.c[0] = x.c[1] = x.c[2] = 0.f;
  x.m[0] = x.m[1] = x.m[2] = 0.f;
  x.z = make_uint4(0, 0, 0, 0);
  // look-ahead indices run past S (in 64-bit, so they cannot wrap)
  x.in = s64 >= 0 && s64 < S;
  if (!x.in) return x;
  const int s = static_cast<int>(s64);
  if (MODE == 0) {
    x.a[0] = dirs[3 * static_cast<int64_t>(s)];
    x.a[1] = dirs[3 * static_cast<int64_t>(s) + 1];
    x.a[2] = dirs[3 * static_cast<int64_t>(s) + 2];
  } else {
    x.in = radius[s] > 0;
    x.a[0] = means[s]; x.a[1] = means[S + s]; x.a[2] = means[2 * S + s];
  }
  if (g < 2) x.z = *reinterpret_cast<const uint4*>(latents + static_cast<int64_t>(s / per) * 16 + 8 * g);
  if (BWD && g == 0) {
#pragma unroll
    for (int i = 0; i < kMlpOut; ++i) {
      x.c[i] = dL_dc[(MODE == 1 ? 6 + i : i) * cs + s * ss];
      if (MODE == 1 && dmean) x.m[i] = dmean[static_cast<int64_t>(i) * S + s];
    }
  }
  return x;
}

// Unit view direction of a loaded sample (MODE 1: from the mean and camera).
template <int MODE>
__device__ __forceinline__ void sample_dir(const SampleIn& x, const DevCam& cam, float d[3], float& len) {
  len = 1.f;
  if (MODE == 0) {
    d[0] = x.a[0]; d[1] = x.a[1]; d[2] = x.a[2];
  } else if (x.in) {
    view_dir(x.a, cam, d, len);
  } else {
    d[0] = 0.f; d[1] = 0.f; d[2] = 1.f;
  }
}

// MODE 0: samples s < S with unit directions dirs[s][3], latent s / per,
//         colours out[s][3].
// MODE 1: sample s = Gaussian s of the projection; direction from its centre
//         and the camera; colours written into the record of every live
//         Gaussian (radius > 0).
template <int MODE>
__global__ __launch_bounds__(256) void k_mlp_fwd(int S, int per, const uint16_t* __restrict__ latents,
                                                 const float* __restrict__ dirs, const float* __restrict__ means,
                                                 const int* __restrict__ radius, DevCam cam,
                                                 const uint4* __restrict__ ops, const float* __restrict__ bias,
                                                 float* __restrict__ out, float* __restrict__ records) {
  __shared__ MlpShared sh;
  load_packed(sh, ops, bias);
  __syncthreads();
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
  const int stride = gridDim.x * 4;
  int grp = blockIdx.x * 4 + wave;
  SampleIn cur = load_sample<MODE, false>(static_cast<int64_t>(grp) * 16 + r, S, per, g, latents, dirs, means, radius,
                                          nullptr);
  for (; static_cast<int64_t>(grp) * 16 < S; grp += stride) {
    const int s = grp * 16 + r;
    const SampleIn nxt = load_sample<MODE, false>((static_cast<int64_t>(grp) + stride) * 16 + r, S, per, g, latents,
                                                  dirs, means, radius, nullptr);
    const bool valid = cur.in;
    float d[3], len;
    sample_dir<MODE>(cur, cam, d, len);
    MlpFwdState st;
    st.X = input_operand(g, valid, cur.z, d);
    mlp_forward_group<false>(sh, lane, st);
    cur = nxt;
    if (g == 0 && valid) {
#pragma unroll
      for (int i = 0; i < kMlpOut; ++i) {
        float c = sigmoidf(st.o[i] + sh.bias[128 + i]);
        c = isfinite(c) ? c : 0.0f;
        if (MODE == 0) out[3 * s + i] = c;
        else records[12 * static_cast<int64_t>(s) + 6 + i] = c;
      }
    }
  }
}

// At least four groups of 16 per wave; about three workgroups per CU at most
// (each copies the 31 KB operand image to LDS once).
static unsigned mlp_grid(int64_t S) {
  return static_cast<unsigned>(std::max<int64_t>(1, std::min<int64_t>(ceil_div(S, 256), 768)));
}

gs_status launch_mlp_pack(const uint16_t* params, void* packed, hipStream_t s) {
  uint4* ops = static_cast<uint4*>(packed);
  float* bias = reinterpret_cast<float*>(ops + kOps * 64);
  { TimedLaunch gs_tl("k_mlp_pack", s); k_mlp_pack<<<kOps, 64, 0, s>>>(params, ops, bias); }
  return check_launch("k_mlp_pack");
}

static const uint4* packed_ops(const void* p) { return static_cast<const uint4*>(p); }
static const float* packed_bias(const void* p) {
  return reinterpret_cast<const float*>(static_cast<const uint4*>(p) + kOps * 64);
}

gs_status launch_mlp_fwd(int64_t S, int per, const uint16_t* latents, const float* dirs, const void* packed,
                         float* rgb, hipStream_t s) {
  if (S == 0) return GS_OK;
  DevCam dummy{};
  { TimedLaunch gs_tl("k_mlp_fwd<0>", s); k_mlp_fwd<0><<<mlp_grid(S), 256, 0, s>>>(static_cast<int>(S), per, latents, dirs, nullptr, nullptr, dummy,
                                           packed_ops(packed), packed_bias(packed), rgb, nullptr); }
  return check_launch("k_mlp_fwd");
}

gs_status launch_mlp_render(int64_t n, const uint16_t* latents, const float* means, const int* radius,
                            const DevCam& cam, const void* packed, float* records, hipStream_t s) {
  if (n == 0) return GS_OK;
  { TimedLaunch gs_tl("k_mlp_fwd<1>", s); k_mlp_fwd<1><<<mlp_grid(n), 256, 0, s>>>(static_cast<int>(n), 1, latents, nullptr, means, radius, cam,
                                           packed_ops(packed), packed_bias(packed), nullptr, records); }
  return check_launch("k_mlp_render");
}

size_t mlp_packed_bytes() { return kOps * 64 * sizeof(uint4) + kBiasFloats * sizeof(float); }


// ------------------------------------------------------------------ backward
//
// A wave takes groups of 16 samples in the forward's lane layout, recomputes
// the forward (keeping the pre-activations for the ReLU masks) and runs
//   g3 = dL/dc * c (1 - c)            (quarter-0 lanes, rows 0..2)
//   g2 = (W3^T g3) [a2 > 0],  g1 = (W2^T g2) [a1 > 0],  dx = W1^T g1
// with the packed transposed weights as A operands, so every gradient lands in
// the D layout like the activations.  dx rows 0..15 are dL/dz, rows 16..31
// dL/dY (the SH encoding), which the basis gradient carries to the direction.
// The gradients entering the transposed products are hi + lo BF16 pairs as in
// the forward.  Weight gradients contract over samples:
//   dW1 += g1 x^T,  dW2 += g2 h1^T,  dW3 += g3 h2^T
// as hi.hi + lo.hi + hi.lo (the lo.lo term, about 2^-18 relative, is dropped).
// A lane of those operands holds four samples of one unit, where the layers
// above leave four units of one sample: the operands go to LDS as they are
// ([sample][unit], four units a store) and come back through the transposing LDS
// read.  Two waves share the sums of dW1 and dW2: after a barrier each takes half
// of the tiles over both waves' samples (32, a whole K), so that a wave's sums
// take 64 registers and not 112 and two waves fit a SIMD without spills.  dW3 (3 of
// 16 rows used) stays with the wave, K running over its 16 samples twice:
// [g_hi | g_hi] x [h_hi | h_lo], then [g_lo | 0] x [h_hi | h_lo].  Sums stay in
// registers for the wave's whole share; a workgroup adds its waves' up in LDS and
// writes one partial vector, and a fixed-order sum over workgroups makes the
// result deterministic for a given sample count.

constexpr int kPartStride = GS_MLP_PARAMS + 1;  // parameters, then the loss
constexpr int kBwdWaves = 8;                     // waves of a workgroup
constexpr int kBwdGroupsMax = 256;               // workgroups: one per CU, whose LDS it takes

// The hi and lo operands of two groups staged at m0 and m1: slots 0..3 hold the
// first group's samples, 4..7 the second's.
struct PairOp {
  bf16x8 hi, lo;
};
template <int ROW>
__device__ __forceinline__ PairOp stage_pair(const __bf16 (*m0)[16][ROW], const __bf16 (*m1)[16][ROW], int b, int g, int r) {
  PairOp o;
  o.hi = join(stage_get<ROW>(m0[0], b, g, r), stage_get<ROW>(m1[0], b, g, r));
  o.lo = join(stage_get<ROW>(m0[1], b, g, r), stage_get<ROW>(m1[1], b, g, r));
  return o;
}

__device__ __forceinline__ floatx4 mfma32(const bf16x8& a, const bf16x8& b, const floatx4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ floatx4 mfma_dw(const PairOp& a, const PairOp& b, const floatx4& c) {
  return mfma32(a.hi, b.lo, mfma32(a.lo, b.hi, mfma32(a.hi, b.hi, c)));
}

// Sum over the 16 lanes of each DPP row (the 16 samples of one quarter); every
// lane of the row gets the sum.  Fixed order, so deterministic.
__device__ __forceinline__ float row_sum16(float v) {
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, false));   // quad 1,0,3,2
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, false));   // quad 2,3,0,1
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x124, 0xF, 0xF, false));  // row_ror 4
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xF, 0xF, false));  // row_ror 8
  return v;
}

__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// A wave's sums: rows 32 half .. + 31 of dW1 and dW2 over its pair's samples, the
// rest over its own.
struct MlpGrads {
  floatx4 dW1[2][2], dW2[2][4], dW3[4];
  float db1[16], db2[16], db3[3], loss;
};

// One group: forward, loss gradient, backward, weight-gradient update (every wave
// of the workgroup at once: it has two barriers).  Returns dL/dz (dxz) and dL/dY
// (dxe) of this lane's sample in the D layout.
//
// Latency bounds it, with LDS (the packed tiles, 30 KB a group, and the staged
// operands: two fifths of the cycles), VALU issue (530 instructions a group, half)
// and the matrix cores (98 products, a quarter) all busy: 150 us for 1,048,576
// samples, 64 to a latent.  One wave per SIMD with all 112 registers of sums and
// 16-bit transposing stores took 260; two whole waves per SIMD, which spill, 190; a
// pair of groups in lockstep by one wave per SIMD 220.
template <int MODE, class Prefetch>
__device__ __forceinline__ void mlp_bwd_group(const MlpShared& sh, MlpStage* stage, int wave, MlpGrads& G, int lane,
                                              const SampleIn& x, const float d[3], bool loss_mode, float scale,
                                              floatx4& dxz, floatx4& dxe, const Prefetch& prefetch) {
  const int g = lane >> 4, r = lane & 15;
  const bool valid = x.in;
  const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
  MlpStage& sg = stage[wave];
  MlpFwdState st;
  st.X = input_operand(g, valid, x.z, d);
  lds_barrier();   // the pair's reads of the group before
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const bf16x4 hi = {st.X.hi[4 * q], st.X.hi[4 * q + 1], st.X.hi[4 * q + 2], st.X.hi[4 * q + 3]};
    const bf16x4 lo = {st.X.lo[4 * q], st.X.lo[4 * q + 1], st.X.lo[4 * q + 2], st.X.lo[4 * q + 3]};
    __builtin_memcpy(&sg.x[0][r][8 * g + 4 * q], &hi, sizeof(hi));
    __builtin_memcpy(&sg.x[1][r][8 * g + 4 * q], &lo, sizeof(lo));
  }
  mlp_forward_group<true>(sh, lane, st, &sg);
  uint4 w[8];
  tiles<4>(sh, kOpW3T, lane, w);
  floatx4 g3 = zero;
  if (g == 0 && valid) {
#pragma unroll
    for (int i = 0; i < kMlpOut; ++i) {
      const float c = sigmoidf(st.o[i] + sh.bias[128 + i]);
      float gc;
      if (MODE == 0 && loss_mode) {
        const float e = c - x.c[i];
        G.loss += scale * e * e;
        gc = 2.0f * scale * e;
      } else {
        gc = x.c[i];
      }
      g3[i] = gc * c * (1.0f - c);
      G.db3[i] += g3[i];
    }
  }
  Split8 Bg3;
#pragma unroll
  for (int e = 0; e < 8; e += 2)
    split_put2(Bg3, e, (g == 0 && e < 4) ? g3[e & 3] : 0.0f, (g == 0 && e < 4) ? g3[(e & 3) + 1] : 0.0f);
  if (g == 0) {
    const bf16x4 hi = {Bg3.hi[0], Bg3.hi[1], Bg3.hi[2], Bg3.hi[3]}, lo = {Bg3.lo[0], Bg3.lo[1], Bg3.lo[2], Bg3.lo[3]};
    __builtin_memcpy(&sg.g3[0][r][0], &hi, sizeof(hi));
    __builtin_memcpy(&sg.g3[1][r][0], &lo, sizeof(lo));
  }
  stage_fence();
  {
    const bf16x4 hi = stage_get<kRowG3>(sg.g3[0], 0, g, r), lo = stage_get<kRowG3>(sg.g3[1], 0, g, r);
    const bf16x8 hh = join(hi, hi), l0 = join(lo, bf16x4{});
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const bf16x8 h = join(stage_get<kRow>(sg.hg2[0], b, g, r), stage_get<kRow>(sg.hg2[1], b, g, r));
      G.dW3[b] = mfma32(l0, h, mfma32(hh, h, G.dW3[b]));
    }
  }
  floatx4 t2[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const floatx4 t = mfma2(w[b], Bg3, zero);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      t2[b][i] = __builtin_amdgcn_inverse_ballot_w64(st.m2.m[b][i]) ? t[i] : 0.0f;
      G.db2[4 * b + i] += t2[b][i];
    }
  }
  tiles<8>(sh, kOpW2T, lane, w);
  Split8 G0, G1;
  d_to_b(t2, G0, G1);
  stage_fence();
  stage_put(sg.hg2, g, r, G0, G1);
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const floatx4 t = mfma2(w[2 * b + 1], G1, mfma2(w[2 * b], G0, zero));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      t2[b][i] = __builtin_amdgcn_inverse_ballot_w64(st.m1.m[b][i]) ? t[i] : 0.0f;
      G.db1[4 * b + i] += t2[b][i];
    }
  }
  tiles<MODE == 1 ? 4 : 2>(sh, kOpW1T, lane, w);
  Split8 H0, H1;
  d_to_b(t2, H0, H1);
  stage_put(sg.g1, g, r, H0, H1);
  dxz = mfma2(w[1], H1, mfma2(w[0], H0, zero));
  if (MODE == 1) dxe = mfma2(w[3], H1, mfma2(w[2], H0, zero));
  prefetch();   // the next group's inputs
  lds_barrier();
  const MlpStage &s0 = stage[wave & ~1], &s1 = stage[wave | 1];
  const int half = 2 * (wave & 1);
  {
    PairOp h[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) h[b] = stage_pair<kRow>(s0.h1, s1.h1, b, g, r);
#pragma unroll
    for (int bo = 0; bo < 2; ++bo) {
      const PairOp a = stage_pair<kRow>(s0.hg2, s1.hg2, half + bo, g, r);
#pragma unroll
      for (int bi = 0; bi < 4; ++bi) G.dW2[bo][bi] = mfma_dw(a, h[bi], G.dW2[bo][bi]);
    }
  }
  // the latent inputs are BF16: their lo part is zero
  const PairOp x1 = stage_pair<kRowX>(s0.x, s1.x, 1, g, r);
  const bf16x8 x0 = join(stage_get<kRowX>(s0.x[0], 0, g, r), stage_get<kRowX>(s1.x[0], 0, g, r));
#pragma unroll
  for (int bo = 0; bo < 2; ++bo) {
    const PairOp a = stage_pair<kRow>(s0.g1, s1.g1, half + bo, g, r);
    G.dW1[bo][0] = mfma32(a.lo, x0, mfma32(a.hi, x0, G.dW1[bo][0]));
    G.dW1[bo][1] = mfma_dw(a, x1, G.dW1[bo][1]);
  }
}

// MODE 0: sample s has direction dirs[s] and latent s / per (per a power of
//         two); dL/dc from dL_dc[S][3], or, with target != NULL, from the
//         distillation loss scale * |c - target|^2 (accumulated into the
//         partial's last slot).  dlat[S / per][16] is overwritten.
// MODE 1: sample s = Gaussian s of the projection (per = 1), dL/dc from rows
//         6..8 of g2d[9][S] or entries 6..8 of the accumulator rows (cs, ss:
//         see load_sample); dlat[s] and the direction's share of dL/dmean are
//         written for live Gaussians (dmean is added to), zeros elsewhere.
template <int MODE>
__global__ __launch_bounds__(64 * kBwdWaves) void k_mlp_bwd(int S, int per, const uint16_t* __restrict__ latents,
                                                 const float* __restrict__ dirs, const float* __restrict__ means,
                                                 const int* __restrict__ radius, DevCam cam,
                                                 const uint4* __restrict__ ops, const float* __restrict__ bias,
                                                 const float* __restrict__ dL_dc, const float* __restrict__ target,
                                                 float scale, float* __restrict__ dlat, float* __restrict__ dmean,
                                                 float* __restrict__ partial, int64_t cs, int64_t ss) {
  __shared__ MlpShared sh;
  __shared__ union {
    MlpStage stage[kBwdWaves];
    float part[2][kPartStride];
  } u;
  load_packed(sh, ops, bias);
  __syncthreads();
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
  const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
  MlpGrads G;
#pragma unroll
  for (int b = 0; b < 4; ++b) { G.dW2[0][b] = zero; G.dW2[1][b] = zero; G.dW3[b] = zero; }
#pragma unroll
  for (int b = 0; b < 2; ++b) { G.dW1[0][b] = zero; G.dW1[1][b] = zero; }
#pragma unroll
  for (int k = 0; k < 16; ++k) { G.db1[k] = 0.f; G.db2[k] = 0.f; }
  G.db3[0] = G.db3[1] = G.db3[2] = 0.f;
  G.loss = 0.f;

  const int wave_id = blockIdx.x * kBwdWaves + wave, nwaves = gridDim.x * kBwdWaves;
  const int ngroups = (S + 15) / 16;
  // per >= 16: a wave owns whole latents (per / 16 consecutive groups each)
  const int gpl = per >= 16 ? per / 16 : 1;
  const int nunits = ngroups / gpl;
  const bool loss_mode = (MODE == 0) && target != nullptr;
  const float* cin = (MODE == 0 && loss_mode) ? target : dL_dc;
  // groups of this wave in order: units wave_id, wave_id + nwaves, ..., each
  // unit's gpl groups in turn; the next group's inputs are loaded ahead
  auto group_of = [&](int unit, int q) { return (static_cast<int64_t>(unit) * gpl + q) * 16 + r; };
  SampleIn cur = load_sample<MODE, true>(group_of(wave_id, 0), wave_id < nunits ? S : 0, per, g, latents, dirs,
                                         means, radius, cin, dmean, cs, ss);
  // a pair of waves with no unit at all (few units, one step) takes its barriers only
  // (16 samples 17 -> 11 us a call, 64 of one latent 28 -> 19; scalar, so that the
  // branch round the barriers is one)
  const bool idle = uniform(wave_id & ~1) >= nunits;
  if (idle)
    for (int q = 0; q < 2 * gpl; ++q) lds_barrier();
  // (every other wave of a workgroup takes as many steps as its first)
  for (int unit = idle ? nunits + wave : wave_id; unit - wave < nunits; unit += nwaves) {
    floatx4 zacc = zero;
    for (int q = 0; q < gpl; ++q) {
      // MODE 1: addresses that depend on the lane are worked out anew each time;
      // kept across the loop they spill, and a reload waits for the prefetched
      // inputs (70 us against 58 for 200,000 Gaussians)
      int lane = threadIdx.x & 63;
      if constexpr (MODE == 1) asm volatile("" : "+v"(lane));
      const int g = lane >> 4, r = lane & 15;
      auto group_of = [&](int unit, int q) { return (static_cast<int64_t>(unit) * gpl + q) * 16 + r; };
      const int64_t s = group_of(unit, q);
      const int nunit = (q + 1 < gpl) ? unit : unit + nwaves;
      const int nq = (q + 1 < gpl) ? q + 1 : 0;
      SampleIn nxt;
      const bool valid = cur.in;
      float d[3], len;
      sample_dir<MODE>(cur, cam, d, len);
      floatx4 dxz, dxe;
      mlp_bwd_group<MODE>(sh, u.stage, wave, G, lane, cur, d, loss_mode, scale, dxz, dxe, [&] {
        nxt = load_sample<MODE, true>(group_of(nunit, nq), nunit < nunits ? S : 0, per, g, latents, dirs, means, radius,
                                      cin, dmean, cs, ss);
      });
      if (per >= 16) {
#pragma unroll
        for (int i = 0; i < 4; ++i) zacc[i] += row_sum16(dxz[i]);
      } else if (s < S) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float v = dxz[i];
          for (int w = 1; w < per; w <<= 1) v += __shfl_xor(v, w, 16);
          if ((r & (per - 1)) == 0) dlat[s / per * 16 + 4 * g + i] = valid ? v : 0.0f;
        }
      }
      if (MODE == 1) {
        // dL/dd = sum_j dL/dY_j grad Y_j(d); this lane holds j = 4g + i
        float w16[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) w16[j] = ((j >> 2) == g) ? dxe[j & 3] : 0.0f;
        float gd[3];
        sh_basis_vjp(3, d[0], d[1], d[2], w16, gd[0], gd[1], gd[2]);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          gd[k] += __shfl_xor(gd[k], 16, 64);
          gd[k] += __shfl_xor(gd[k], 32, 64);
        }
        if (g == 0 && valid) {
          // d = v / |v| with v = mean - centre:  dL/dv = (dL/dd - d (d . dL/dd)) / |v|
          const float dd = d[0] * gd[0] + d[1] * gd[1] + d[2] * gd[2];
          const float il = __builtin_amdgcn_rcpf(len);
#pragma unroll
          for (int k = 0; k < 3; ++k) dmean[static_cast<int64_t>(k) * S + s] = cur.m[k] + (gd[k] - d[k] * dd) * il;
        }
      }
      cur = nxt;
    }
    if (per >= 16 && r == 0 && unit < nunits) {
#pragma unroll
      for (int i = 0; i < 4; ++i) dlat[static_cast<int64_t>(unit) * 16 + 4 * g + i] = zacc[i];
    }
  }

  // the workgroup's partial vector (D layout: row 4g + i of a 16-row block,
  // column r): waves 0..3 and 4..7 add up in turn, each half in its own copy
  // (the first `used` only: the others had no unit, nor had their pair)
  const int used = max(2, min(kBwdWaves, (nunits - static_cast<int>(blockIdx.x) * kBwdWaves + 1) & ~1));
  float* const out = u.part[wave >> 2];
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      G.db1[4 * b + i] = row_sum16(G.db1[4 * b + i]);
      G.db2[4 * b + i] = row_sum16(G.db2[4 * b + i]);
    }
#pragma unroll
  for (int i = 0; i < kMlpOut; ++i) G.db3[i] = row_sum16(G.db3[i]);
  G.loss = row_sum16(G.loss);
  for (int w = 0; w < 4; ++w) {
    __syncthreads();
    if ((wave & 3) != w || uniform(wave) >= used) continue;
    auto add = [&](int p, float v) { out[p] = w ? out[p] + v : v; };
    auto add_half = [&](int p, float v) { out[p] = w > 1 ? out[p] + v : v; };   // rows that every other wave has
#pragma unroll
    for (int bo = 0; bo < 2; ++bo)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int o = 32 * (wave & 1) + 16 * bo + 4 * g + i;
#pragma unroll
        for (int bi = 0; bi < 4; ++bi) add_half(P_W2 + o * kMlpH + 16 * bi + r, G.dW2[bo][bi][i]);
        add_half(P_W1 + o * kMlpIn + r, G.dW1[bo][0][i]);
        add_half(P_W1 + o * kMlpIn + 16 + r, G.dW1[bo][1][i]);
      }
#pragma unroll
    for (int bi = 0; bi < 4; ++bi)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int o = 4 * g + i;
        if (o < kMlpOut) add(P_W3 + o * kMlpH + 16 * bi + r, G.dW3[bi][i]);
      }
    if (r == 0) {
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          add(P_B1 + 16 * b + 4 * g + i, G.db1[4 * b + i]);
          add(P_B2 + 16 * b + 4 * g + i, G.db2[4 * b + i]);
        }
    }
    if (lane == 0) {
#pragma unroll
      for (int i = 0; i < kMlpOut; ++i) add(P_B3 + i, G.db3[i]);
      add(GS_MLP_PARAMS, G.loss);
    }
  }
  __syncthreads();
  for (int p = threadIdx.x; p < kPartStride; p += 64 * kBwdWaves)
    partial[static_cast<int64_t>(blockIdx.x) * kPartStride + p] = used > 4 ? u.part[0][p] + u.part[1][p] : u.part[0][p];
}

// Sum of the workgroups' partial vectors: a block takes 64 parameters, eight
// interleaved sub-sums each, combined in a fixed order.
__global__ __launch_bounds__(512) void k_mlp_reduce(const float* __restrict__ partial, int count,
                                                    float* __restrict__ dparams, float* __restrict__ loss) {
  __shared__ float part[8][64];
  const int t = threadIdx.x & 63, q = threadIdx.x >> 6, p = blockIdx.x * 64 + t;
  float acc = 0.f;
  if (p < kPartStride) {
#pragma unroll 8
    for (int w = q; w < count; w += 8) acc += partial[static_cast<int64_t>(w) * kPartStride + p];
  }
  part[q][t] = acc;
  __syncthreads();
  if (q != 0 || p >= kPartStride) return;
#pragma unroll
  for (int k = 1; k < 8; ++k) acc += part[k][t];
  if (p < GS_MLP_PARAMS) dparams[p] = acc;
  else if (loss) *loss = acc;
}

// Workgroups of the backward for S samples: a unit (a group of 16 samples, or
// the groups of one latent) per wave, up to one workgroup per CU.
static int mlp_bwd_groups(int64_t S, int per) {
  const int64_t groups = std::max<int64_t>(1, ceil_div(S, 16));
  const int64_t units = per >= 16 ? std::max<int64_t>(1, groups / (per / 16)) : groups;
  return static_cast<int>(std::min<int64_t>(kBwdGroupsMax, ceil_div(units, kBwdWaves)));
}

size_t mlp_bwd_workspace(int64_t S, int per) {
  return static_cast<size_t>(mlp_bwd_groups(S, per)) * kPartStride * sizeof(float);
}

static gs_status reduce_partials(const float* ws, int count, float* dparams, float* loss, hipStream_t s) {
  { TimedLaunch gs_tl("k_mlp_reduce", s); k_mlp_reduce<<<static_cast<unsigned>(ceil_div(kPartStride, 64)), 512, 0, s>>>(ws, count, dparams, loss); }
  return check_launch("k_mlp_reduce");
}

gs_status launch_mlp_bwd(int64_t S, int per, const uint16_t* latents, const float* dirs, const void* packed,
                         const float* dL_drgb, const float* target, float scale, float* dlat, float* dparams,
                         float* loss, void* ws, hipStream_t s) {
  const int groups = mlp_bwd_groups(S, per);
  DevCam dummy{};
  { TimedLaunch gs_tl("k_mlp_bwd<0>", s); k_mlp_bwd<0><<<groups, 64 * kBwdWaves, 0, s>>>(static_cast<int>(S), per, latents, dirs, nullptr, nullptr, dummy,
                                         packed_ops(packed), packed_bias(packed), dL_drgb, target, scale, dlat,
                                         nullptr, static_cast<float*>(ws), 1, 3); }
  gs_status st = check_launch("k_mlp_bwd");
  if (st != GS_OK) return st;
  return reduce_partials(static_cast<float*>(ws), groups, dparams, loss, s);
}

gs_status launch_mlp_render_bwd(int64_t n, const uint16_t* latents, const float* means, const int* radius,
                                const DevCam& cam, const void* packed, const float* g2d, bool rows, float* dlat,
                                float* dmeans, float* dparams, void* ws, hipStream_t s) {
  const int groups = mlp_bwd_groups(n, 1);
  const int64_t cs = rows ? 1 : n, ss = rows ? kAccStride : 1;
  { TimedLaunch gs_tl("k_mlp_bwd<1>", s); k_mlp_bwd<1><<<groups, 64 * kBwdWaves, 0, s>>>(static_cast<int>(n), 1, latents, nullptr, means, radius, cam,
                                         packed_ops(packed), packed_bias(packed), g2d, nullptr, 0.0f, dlat, dmeans,
                                         static_cast<float*>(ws), cs, ss); }
  gs_status st = check_launch("k_mlp_render_bwd");
  if (st != GS_OK) return st;
  return reduce_partials(static_cast<float*>(ws), groups, dparams, nullptr, s);
}

// ------------------------------------------------------------------ training support

// SH colour of Gaussian s / per at direction dirs[s] (the projection's colour
// rule at an arbitrary direction), optionally clamped to [0, 1].
__global__ __launch_bounds__(256) void k_sh_colour(int S, int per, int n, int deg, const float* __restrict__ sh,
                                                   const float* __restrict__ dirs, int clamp01,
                                                   float* __restrict__ out) {
  const int s = blockIdx.x * 256 + threadIdx.x;
  if (s >= S) return;
  const int i = s / per;
  float Y[16];
  sh_basis(deg, dirs[3 * s], dirs[3 * s + 1], dirs[3 * s + 2], Y);
  const int nc = (deg + 1) * (deg + 1);
  for (int c = 0; c < 3; ++c) {
    float acc = 0.f;
    for (int j = 0; j < nc; ++j) acc += Y[j] * sh[(static_cast<int64_t>(j) * 3 + c) * n + i];
    float v = fmaxf(acc + 0.5f, 0.0f);
    if (clamp01) v = fminf(v, 1.0f);
    out[3 * static_cast<int64_t>(s) + c] = v;
  }
}

gs_status launch_sh_colour(int64_t S, int per, int64_t n, int deg, const float* sh, const float* dirs, int clamp01,
                           float* out, hipStream_t s) {
  if (S == 0) return GS_OK;
  { TimedLaunch gs_tl("k_sh_colour", s); k_sh_colour<<<static_cast<unsigned>(ceil_div(S, 256)), 256, 0, s>>>(static_cast<int>(S), per, static_cast<int>(n),
                                                                      deg, sh, dirs, clamp01, out); }
  return check_launch("k_sh_colour");
}

// Adam (bias-corrected), FP32 master parameters, optional BF16 copy rounded to
// nearest even for the forward.
__global__ __launch_bounds__(256) void k_adam(int64_t n, float* __restrict__ p, const float* __restrict__ grad,
                                              float* __restrict__ m, float* __restrict__ v,
                                              uint16_t* __restrict__ pb, float lr, float b1, float b2, float eps,
                                              float bc1, float bc2) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i >= n) return;
  const float gi = grad[i];
  const float mi = b1 * m[i] + (1.0f - b1) * gi;
  const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float pi = p[i] - lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
  p[i] = pi;
  if (pb) {
    const __bf16 h = static_cast<__bf16>(pi);
    uint16_t bits;
    __builtin_memcpy(&bits, &h, sizeof(bits));
    pb[i] = bits;
  }
}

gs_status launch_adam(int64_t n, float* p, const float* g, float* m, float* v, uint16_t* pb, float lr, float b1,
                      float b2, float eps, float bc1, float bc2, hipStream_t s) {
  if (n == 0) return GS_OK;
  { TimedLaunch gs_tl("k_adam", s); k_adam<<<static_cast<unsigned>(ceil_div(n, 256)), 256, 0, s>>>(n, p, g, m, v, pb, lr, b1, b2, eps, bc1, bc2); }
  return check_launch("k_adam");
}

}  // namespace gs
