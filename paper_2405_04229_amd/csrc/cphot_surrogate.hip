// Transport surrogate: training-set generation with the exact layered tracer,
// output normalisation, training (forward + backward on bf16 matrix cores with
// FP32 accumulation, Adam on FP32 master weights) and batch inference.
//
// The surrogate replaces the layered tracer's correction to the straight line
// (the role of the thesis's precomputed correction table, Sec. 4.4.1) by a
// small network trained on photons the exact tracer generates: over planar
// layers, or over the spherical shells of a curved Earth (Sec. 3.3.4).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "cphot_device.h"
#include "cphot_internal.h"
#include "cphot_mlp.h"
#include "cphot_walk64.h"

namespace cphot {

namespace {

constexpr int kTrainWave = 64;  // samples per training block

__device__ __forceinline__ f32x4 zero4() { return f32x4{0.f, 0.f, 0.f, 0.f}; }

// ---------------------------------------------------------------------------- training set

struct TrainSetParams {
  float4 const* layers;
  float4 const* moments;  // closed-form layer-sum moments [obs][j][5] (planar targets)
  float2 const* lambins;
  int n_layers, n_lam;
  int geometry;  // CPHOT_SURROGATE_PLANAR | CPHOT_SURROGATE_CURVED
  double earth_radius;
  float dh, lam_min, lam_max;
  float lo[5], hi[5];
  uint32_t key0, key1;
  int64_t first, n;
  float* X;
  float* Y;
};

// Inputs of a sample: start boundary (index), cos zenith, azimuth, wavelength bin,
// observation level.
struct SampleInput {
  float h_obs, ct, phi;
  uint32_t start_bin;  // start layer + 256 wavelength bin
};

__device__ __forceinline__ SampleInput sample_input(const TrainSetParams& p, uint64_t i) {
  const uint4 w = philox((uint32_t)i, 0u, (uint32_t)(i >> 32), TAG_TRAIN, p.key0, p.key1);
  const uint4 v = philox((uint32_t)i, 1u, (uint32_t)(i >> 32), TAG_TRAIN, p.key0, p.key1);
  SampleInput in;
  in.h_obs = p.lo[4] + (p.hi[4] - p.lo[4]) * u24(w.x);
  // start: the lower boundary of a layer (shell) above the observation layer, drawn
  // uniformly among those in the box (integer arithmetic on the word's top 24 bits);
  // inside its start layer a photon is straight, so the network learns the
  // correction from that boundary on, a smooth function of the boundary height
  const int j_obs = (int)floorf(in.h_obs / p.dh);
  const int j_lo = max((int)ceilf(p.lo[0] / p.dh), j_obs + 1);
  const int j_hi = (int)floorf(p.hi[0] / p.dh);
  const int m = max(j_hi - j_lo + 1, 1);
  const int jj = j_lo + (int)(((uint64_t)(w.y >> 8) * (uint64_t)m) >> 24);
  in.ct = p.lo[1] + (p.hi[1] - p.lo[1]) * u24(w.z);
  in.phi = p.lo[2] + (p.hi[2] - p.lo[2]) * u24(w.w);
  const int kb = min((int)floorf(u24(v.x) * (float)p.n_lam), p.n_lam - 1);
  in.start_bin = (uint32_t)jj + ((uint32_t)kb << 8);
  return in;
}

// Curved targets: by the spherical symmetry the start is above the Earth point (0, 0);
// the chord from there to the sphere R + h_obs and the walk, in FP64, per metre of chord
// (the absolute quantities grow with the slant distance).
__device__ __forceinline__ float4 curved_target(const TrainSetParams& p, const double2* s_n, const float4* s_lay,
                                                float2 sp, double he, const SampleInput& in) {
  const double Re = p.earth_radius, ho = in.h_obs, ct = in.ct;
  double s_ch, psi_s;
  chord_f64(Re, ho, he, ct, s_ch, psi_s);
  Walk64 w;
  if (!shell_descent_f64(s_n, s_lay, (double)p.dh, p.n_layers, ho, Re, he, ct, w) &&
      !shell_walk_f64(s_lay, (double)p.dh, p.n_layers, ho, Re, he, ct, w)) {
    const float q = __builtin_nanf("");
    return make_float4(q, q, q, q);
  }
  const double tau = (double)sp.x * w.tR + (double)sp.y * w.tA;
  // the offset across the plane of the start direction is zero by symmetry
  return make_float4((float)((w.across - psi_s) * (Re + ho) / s_ch), 0.f, (float)(((w.len - s_ch) + w.opt) / s_ch),
                     (float)(-tau / s_ch));
}

// a / b of normal floats, off the rounded quotient by 2^-20 of a unit in the last place: the
// hardware's reciprocal (one unit) and the remainder of the quotient it gives. The planar
// targets' errors against 64 bits are those of rounded divisions (offset 2.05e-7 m root mean
// square, 2.10e-7 with the reciprocal alone) at 132 us for 2.2e6 samples (193 and 109 us).
__device__ __forceinline__ float quotient(float a, float b) {
  const float r = __builtin_amdgcn_rcpf(b), q = a * r;
  return fmaf(fmaf(-b, q, a), r, q);
}

// Planar targets: landing offset from the straight line, optical path excess
// sum (n - 1) l + (path - straight path) and -tau, beyond the straight line's own sums.
__device__ __forceinline__ float4 planar_target(const TrainSetParams& p, const float4* s_lay, float2 sp, float h_e,
                                                const SampleInput& in) {
  const int i0 = min((int)(h_e / p.dh), p.n_layers - 1);
  const int iobs = (int)floorf(in.h_obs / p.dh);
  const float s0 = sqrtf((1.f - in.ct) * (1.f + in.ct)), c0 = in.ct, d0 = s_lay[i0].x, ic0 = 1.0f / c0;
  float dr = 0.f, gex = 0.f, opt = 0.f, tau = 0.f;
  // a leg of vertical extent `span` in layer k: beyond the same extent at the start sine,
  // without subtracting nearly equal lengths (s - s0 = -s0 e)
  auto leg = [&](int k, float span, bool last) {
    const float4 L = s_lay[k];
    float s, c2, e;
    layer_angle(s0, c0, d0, L.x, L.y, s, c2, e);
    // cos of this layer: the estimate's last place corrected from its own square
    const float ic = __builtin_amdgcn_rsqf(c2), c1 = c2 * ic, c = fmaf(fmaf(-c1, c1, c2), 0.5f * ic, c1);
    const float path = last ? span / c : span * ic;
    opt = fmaf(L.x, path, opt);
    tau = fmaf(fmaf(L.z, sp.x, L.w * sp.y), path, tau);
    const float dsq = -s0 * e * (s + s0);   // s^2 - s0^2
    const float den = fmaf(s, c0, s0 * c);  // zero only for a vertical photon, whose offset is zero
    if (den > 0.f) dr = fmaf(span, quotient(dsq, den * c * c0), dr);
    gex = fmaf(span, quotient(dsq, c * c0 * (c + c0)), gex);
  };
  float z = h_e;
  for (int i = i0; i > iobs; --i) {
    const float zb = (float)i * p.dh;
    leg(i, z - zb, false);
    z = zb;
  }
  leg(iobs, z - in.h_obs, true);
  // the straight line's own sums from the start boundary down to h_obs (full layers
  // from the moments, the observation layer's span directly): the network learns
  // only what refraction adds to them
  const float4* mr = p.moments + ((size_t)iobs * p.n_layers + i0) * 5;
  const float4 Lo = s_lay[iobs];
  const float top = (float)(iobs + 1) * p.dh - in.h_obs;
  const float opt_s = ic0 * fmaf(Lo.x, top, mr[2].x);
  const float tau_s = ic0 * fmaf(sp.x, mr[2].w, fmaf(sp.y, mr[3].z, fmaf(Lo.z, sp.x, Lo.w * sp.y) * top));
  // along the photon's horizontal direction; zero across it for horizontal layers
  return make_float4(dr, 0.f, (gex + opt) - opt_s, tau_s - tau);
}

// Two samples per thread. Bound by arithmetic, in FP64 over shells: a wave walks as many
// shells as the highest of its starts, 1 to 80. The block's samples are therefore ordered by
// start layer first (a counting sort of their inputs in LDS), so that the lanes of a wave
// walk alike, and each wave takes one group from below and its mirror image from above, so
// that the waves end together.
// 1e6 samples over 80 shells 472 -> 121 us, 2.2e6 over 80 planar layers 274 -> 132 us. Blocks
// of 128 and 512 threads measured within 6 % of this; more waves per SIMD (6, 8) spill in
// the general walk and lose up to half.
constexpr int kSetBlock = 256, kSetSamples = 2 * kSetBlock;
template <bool CURVED>
__global__ __launch_bounds__(kSetBlock, 4) void k_training_set(TrainSetParams p) {
  __shared__ float4 s_lay[kMaxLayers];
  __shared__ double2 s_n[CURVED ? kMaxLayers : 1];  // n - 1 and 1 / n
  __shared__ float2 s_lam[kMaxLambdaBins];
  __shared__ uint32_t s_count[256];  // per start layer; 255: none
  __shared__ SampleInput s_in[kSetSamples];
  __shared__ uint16_t s_of[kSetSamples];  // sample of each place
  const int t = threadIdx.x;
  for (int i = t; i < p.n_layers; i += kSetBlock) {
    s_lay[i] = p.layers[i];
    if constexpr (CURVED) {
      const double d = (double)p.layers[i].x;
      s_n[i] = make_double2(d, 1.0 / (1.0 + d));
    }
  }
  for (int i = t; i < p.n_lam; i += kSetBlock) s_lam[i] = p.lambins[i];
  for (int i = t; i < 256; i += kSetBlock) s_count[i] = 0u;
  __syncthreads();
  const int64_t j0 = (int64_t)blockIdx.x * kSetSamples;
  SampleInput in[2] = {};
  uint32_t key[2] = {255u, 255u}, rank[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int64_t j = j0 + t + q * kSetBlock;
    if (j < p.n) {
      in[q] = sample_input(p, (uint64_t)(p.first + j));
      key[q] = in[q].start_bin & 255u;
      const uint32_t kb = in[q].start_bin >> 8;
      float* x = p.X + 5 * j;
      x[0] = (float)(int)key[q] * p.dh;
      x[1] = in[q].ct;
      x[2] = in[q].phi;
      x[3] = p.lam_min + ((float)(int)kb + 0.5f) * (p.lam_max - p.lam_min) / (float)p.n_lam;
      x[4] = in[q].h_obs;
    }
    rank[q] = atomicAdd(&s_count[key[q]], 1u);
  }
  __syncthreads();
  if (t < 64) {  // first place of each start layer
    uint32_t carry = 0;
    for (int b = t; b < 256; b += 64) {
      const uint32_t v = s_count[b], end = wave_scan_add(v);
      s_count[b] = carry + end - v;
      carry += (uint32_t)__builtin_amdgcn_readlane((int)end, 63);
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const uint32_t place = s_count[key[q]] + rank[q];
    s_in[place] = in[q];
    s_of[place] = (uint16_t)(t + q * kSetBlock);
  }
  __syncthreads();
  // not unrolled: the walks stay in the instruction cache
#pragma nounroll
  for (int q = 0; q < 2; ++q) {
    const int at = q == 0 ? t : kSetSamples - 1 - t;
    const int64_t of = j0 + s_of[at];
    if (of >= p.n) continue;
    const SampleInput si = s_in[at];
    const float2 sp = s_lam[si.start_bin >> 8];
    const float h_e = (float)(int)(si.start_bin & 255u) * p.dh;
    float4 y;
    if constexpr (CURVED) y = curved_target(p, s_n, s_lay, sp, (double)h_e, si);
    else y = planar_target(p, s_lay, sp, h_e, si);
    float* out = p.Y + 4 * of;
    out[0] = y.x;
    out[1] = y.y;
    out[2] = y.z;
    out[3] = y.w;
  }
}

// ---------------------------------------------------------------------------- normalisation

__global__ void k_zero_f64(double* a, int n) {
  if ((int)threadIdx.x < n) a[threadIdx.x] = 0.0;
}

__global__ __launch_bounds__(256) void k_output_sums(const float* __restrict__ Y, int64_t n, double* sums) {
  double s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < n; j += (int64_t)gridDim.x * 256) {
#pragma unroll
    for (int o = 0; o < 4; ++o) {
      const double v = Y[4 * j + o];
      s[o] += v;
      s[4 + o] += v * v;
    }
  }
  __shared__ double red[8][4];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    double v = s[q];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    if (lane == 0) red[q][wid] = v;
  }
  __syncthreads();
  if (threadIdx.x < 8) {
    const double v = red[threadIdx.x][0] + red[threadIdx.x][1] + red[threadIdx.x][2] + red[threadIdx.x][3];
    atomicAdd(sums + threadIdx.x, v);
  }
}

__global__ void k_output_norm(const double* sums, int64_t n, float* norm) {
  const int o = threadIdx.x;
  if (o >= 4) return;
  const double mean = sums[o] / (double)n;
  const double var = sums[4 + o] / (double)n - mean * mean;
  norm[16 + o] = (float)mean;
  norm[20 + o] = (float)sqrt(var > 1e-30 ? var : 1e-30);
}

// ---------------------------------------------------------------------------- packing

struct TrainWeights {  // bf16 operand layouts for the training kernel (k-contiguous)
  __bf16 w1t[64][32];  // [out unit][input k], k >= 5 zero
  __bf16 w2t[64][64];  // [out][in]
  __bf16 w2[64][64];   // [in][out]
  __bf16 w3t[16][64];  // [output o][in], o >= 4 zero
  __bf16 w3[64][32];   // [in][output o], o >= 4 zero
};

// Builds the training layouts and the inference image from the FP32 master
// weights and the normalisation (at creation, after new parameters or a new
// normalisation; a training step updates its own entries, see k_adam).
__global__ __launch_bounds__(256) void k_pack(const float* __restrict__ m, const float* __restrict__ norm,
                                             TrainWeights* tw, MlpImage* im) {
  const int t = blockIdx.x * 256 + threadIdx.x;
  const int T = gridDim.x * 256;
  for (int e = t; e < 64 * 32; e += T) {
    const int o = e / 32, k = e % 32;
    tw->w1t[o][k] = (__bf16)(k < 5 ? m[kOffW1 + k * 64 + o] : 0.f);
  }
  for (int e = t; e < 64 * 64; e += T) {
    const int a = e / 64, b = e % 64;
    tw->w2t[a][b] = (__bf16)m[kOffW2 + b * 64 + a];
    tw->w2[a][b] = (__bf16)m[kOffW2 + a * 64 + b];
  }
  for (int e = t; e < 16 * 64; e += T) {
    const int o = e / 64, i = e % 64;
    tw->w3t[o][i] = (__bf16)(o < 4 ? m[kOffW3 + i * 4 + o] : 0.f);
  }
  for (int e = t; e < 64 * 32; e += T) {
    const int i = e / 32, o = e % 32;
    tw->w3[i][o] = (__bf16)(o < 4 ? m[kOffW3 + i * 4 + o] : 0.f);
  }
  // inference image
  for (int e = t; e < 4 * 64 * 8; e += T) {
    const int mt = e / 512, l = (e / 8) % 64, i = e % 8;
    const int g = l >> 4, c = l & 15;
    im->a1[mt][l][i] = (__bf16)((g == 0 && i < 5) ? m[kOffW1 + i * 64 + 16 * mt + c] : 0.f);
  }
  for (int e = t; e < 4 * 2 * 64 * 8; e += T) {
    const int mt = e / 1024, kt = (e / 512) % 2, l = (e / 8) % 64, i = e % 8;
    const int g = l >> 4, c = l & 15;
    im->a2[mt][kt][l][i] = (__bf16)m[kOffW2 + mlp_unit_of_slot(kt, g, i) * 64 + 16 * mt + c];
  }
  for (int e = t; e < 2 * 64 * 8; e += T) {
    const int kt = e / 512, l = (e / 8) % 64, i = e % 8;
    const int g = l >> 4, c = l & 15;
    im->a3[kt][l][i] = (__bf16)(c < 4 ? m[kOffW3 + mlp_unit_of_slot(kt, g, i) * 4 + c] : 0.f);
  }
  for (int e = t; e < 64; e += T) {
    im->b1[e] = m[kOffB1 + e];
    im->b2[e] = m[kOffB2 + e];
  }
  if (t < 4) im->b3[t] = m[kOffB3 + t];
  if (t < 5) {
    im->in_lo[t] = norm[t];
    im->in_hi[t] = norm[5 + t];
    im->in_scale[t] = norm[10 + t];
  }
  if (t < 4) {
    im->out_mean[t] = norm[16 + t];
    im->out_std[t] = norm[20 + t];
  }
  if (t == 0) im->pad0 = 0.f;
}

// Writes the bf16 copies of parameter i (new FP32 value v) into every slot of the
// training layouts and the inference image that holds it: the inverse of k_pack's
// index maps, so that one Adam thread refreshes its own parameter and a training
// step needs no separate packing pass. Slots that hold zero padding are untouched.
__device__ __forceinline__ void scatter_param(int i, float v, TrainWeights* tw, MlpImage* im) {
  const __bf16 b = (__bf16)v;
  if (i < kOffB1) {  // W1[k][o]
    const int k = i / 64, o = i % 64;
    tw->w1t[o][k] = b;
    im->a1[o / 16][o % 16][k] = b;  // lane c (g = 0) of M-tile o / 16, K slot k
  } else if (i < kOffW2) {
    im->b1[i - kOffB1] = v;
  } else if (i < kOffB2) {  // W2[a][c2]: K slot (kt, g, ii) of unit a, column c2
    const int e = i - kOffW2, a = e / 64, c2 = e % 64;
    tw->w2t[c2][a] = b;
    tw->w2[a][c2] = b;
    const int kt = (a / 16) >> 1, ii = 4 * ((a / 16) & 1) + (a & 3), g = (a % 16) >> 2;
    im->a2[c2 / 16][kt][16 * g + c2 % 16][ii] = b;
  } else if (i < kOffW3) {
    im->b2[i - kOffB2] = v;
  } else if (i < kOffB3) {  // W3[in][o]
    const int e = i - kOffW3, in = e / 4, o = e % 4;
    tw->w3t[o][in] = b;
    tw->w3[in][o] = b;
    const int kt = (in / 16) >> 1, ii = 4 * ((in / 16) & 1) + (in & 3), g = (in % 16) >> 2;
    im->a3[kt][16 * g + o][ii] = b;
  } else {
    im->b3[i - kOffB3] = v;
  }
}

// ---------------------------------------------------------------------------- training step

struct StepParams {
  const float* X;
  const float* Y;
  int64_t n;        // training-set size
  int64_t start;    // first sample of this batch (wraps modulo n)
  int batch;        // samples in the batch (multiple of 64)
  const float* norm;
  const float* master;
  const TrainWeights* tw;
  float* partial;   // [blocks][kMlpParams]
  float* loss_partial;
};

// A row of 64 activations in LDS: padded so that the 16 rows of an operand start in
// different banks.
constexpr int kRow = 72;

// Operand of 16 rows x 32 k from LDS rows (k-contiguous), row l % 16, k = 8 (l / 16) + i.
__device__ __forceinline__ bf16x8 lds_op(const __bf16* rows) {
  const int l = threadIdx.x & 63;
  return *reinterpret_cast<const bf16x8*>(rows + (l & 15) * kRow + (l >> 4) * 8);
}

__device__ __forceinline__ bf16x8 global_op(const __bf16* rows, int ld) {
  const int l = threadIdx.x & 63;
  return *reinterpret_cast<const bf16x8*>(rows + (l & 15) * ld + (l >> 4) * 8);
}

__device__ __forceinline__ bf16x8 zero_op() {
  bf16x8 v;
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = (__bf16)0.f;
  return v;
}

// Four values of a column (rows 4 g .. 4 g + 3), contiguous in the transposed array.
__device__ __forceinline__ void store4(__bf16* at, const __bf16 v[4]) {
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  *reinterpret_cast<bf16x4*>(at) = (bf16x4){v[0], v[1], v[2], v[3]};
}

// Sum of a row of 64 in order.
__device__ __forceinline__ float row_sum(const __bf16* row) {
  float sb = 0.f;
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const bf16x8 v = *reinterpret_cast<const bf16x8*>(row + 8 * q);
#pragma unroll
    for (int i = 0; i < 8; ++i) sb += (float)v[i];
  }
  return sb;
}

// 64 samples on four waves: forward, loss, backward; writes this block's share of
// the gradient of mean((y_hat - t_hat)^2) over the whole batch. The step is bound by
// latency (a chain of five small products, 64 blocks at the usual batch): a wave carries
// 16 samples through all layers and back with no block barrier, all weight operands are
// loaded at the start with the samples, and only the weight gradients, whose sums run
// over the 64 samples, meet in one barrier, a quarter of them per wave. Every product
// and sum keeps the order that one wave doing all of it had (15.2 -> 6.5 us, batch 4096).
__global__ __launch_bounds__(256) void k_train_step(StepParams p) {
  __shared__ __attribute__((aligned(16))) __bf16 H1[64][kRow], H1T[64][kRow];
  __shared__ __attribute__((aligned(16))) __bf16 H2[64][kRow], H2T[64][kRow];  // H2: then dZ2
  __shared__ __attribute__((aligned(16))) __bf16 Z2T[64][kRow], Z1T[64][kRow];
  __shared__ __attribute__((aligned(16))) __bf16 XhT[8][kRow], dY[64][8], dYT[4][kRow];
  __shared__ float sq[16][64];  // squared residuals, row 4 (sample / 16) + r, lane
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int g = l >> 4, c = l & 15;
  const float* norm = p.norm;
  const float* m = p.master;
  const TrainWeights* tw = p.tw;
  const int64_t s0 = p.start + (int64_t)blockIdx.x * kTrainWave;
  auto sample = [&](int s) {  // start < n and batch <= n: wraps at most once
    const int64_t j = s0 + s;
    return j < p.n ? j : j - p.n;
  };
  // ---- everything the chain reads from memory
  bf16x8 w1[4], w2t[4][2], w3t[2], w3[4], w2[4][2];
  float b1[4], b2[4], x[5], t[4];
#pragma unroll
  for (int k = 0; k < 5; ++k) x[k] = p.X[5 * sample(16 * w + c) + k];
#pragma unroll
  for (int r = 0; r < 4; ++r) t[r] = p.Y[4 * sample(16 * w + 4 * g + r) + (c & 3)];
#pragma unroll
  for (int nt = 0; nt < 4; ++nt) {
    w1[nt] = global_op(&tw->w1t[16 * nt][0], 32);
    b1[nt] = m[kOffB1 + 16 * nt + c];
  }
#pragma unroll
  for (int nt = 0; nt < 4; ++nt) {
    w2t[nt][0] = global_op(&tw->w2t[16 * nt][0], 64);
    w2t[nt][1] = global_op(&tw->w2t[16 * nt][32], 64);
    b2[nt] = m[kOffB2 + 16 * nt + c];
  }
  w3t[0] = global_op(&tw->w3t[0][0], 64);
  w3t[1] = global_op(&tw->w3t[0][32], 64);
  const float b3 = c < 4 ? m[kOffB3 + c] : 0.f;
  const float mean = norm[16 + (c & 3)], std = norm[20 + (c & 3)];
#pragma unroll
  for (int nt = 0; nt < 4; ++nt) w3[nt] = global_op(&tw->w3[16 * nt][0], 32);
#pragma unroll
  for (int nt = 0; nt < 4; ++nt) {
    w2[nt][0] = global_op(&tw->w2[16 * nt][0], 64);
    w2[nt][1] = global_op(&tw->w2[16 * nt][32], 64);
  }
  // ---- forward, rows = this wave's 16 samples
  bf16x8 xa = zero_op();  // k = 0..4 in the lanes g == 0
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    const __bf16 b = (__bf16)fmaf(x[k] - norm[k], norm[10 + k], -1.0f);
    if (g == 0) {
      xa[k] = b;
      XhT[k][16 * w + c] = b;
    }
  }
  __bf16 h1[4][4], h2[4][4];
#pragma unroll
  for (int nt = 0; nt < 4; ++nt) {
    f32x4 acc = {b1[nt], b1[nt], b1[nt], b1[nt]};
    acc = mfma16(xa, w1[nt], acc);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      h1[nt][r] = (__bf16)fmaxf(acc[r], 0.f);
      H1[16 * w + 4 * g + r][16 * nt + c] = h1[nt][r];
    }
    store4(&H1T[16 * nt + c][16 * w + 4 * g], h1[nt]);
  }
  wave_fence();
  {
    const bf16x8 a0 = lds_op(&H1[16 * w][0]), a1 = lds_op(&H1[16 * w][32]);
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
      f32x4 acc = {b2[nt], b2[nt], b2[nt], b2[nt]};
      acc = mfma16(a0, w2t[nt][0], acc);
      acc = mfma16(a1, w2t[nt][1], acc);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        h2[nt][r] = (__bf16)fmaxf(acc[r], 0.f);
        H2[16 * w + 4 * g + r][16 * nt + c] = h2[nt][r];
      }
      store4(&H2T[16 * nt + c][16 * w + 4 * g], h2[nt]);
    }
  }
  wave_fence();
  {
    f32x4 acc = {b3, b3, b3, b3};
    acc = mfma16(lds_op(&H2[16 * w][0]), w3t[0], acc);
    acc = mfma16(lds_op(&H2[16 * w][32]), w3t[1], acc);
    const float dscale = 2.0f / (4.0f * (float)p.batch);
    __bf16 db[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float d = acc[r] - (t[r] - mean) / std;
      sq[4 * w + r][l] = c < 4 ? d * d : 0.f;
      db[r] = (__bf16)(c < 4 ? d * dscale : 0.f);
      if (c < 8) dY[16 * w + 4 * g + r][c] = db[r];  // outputs 4..7: zero
    }
    if (c < 4) store4(&dYT[c][16 * w + 4 * g], db);
  }
  wave_fence();
  // ---- backward through the layers
  {
    const bf16x8 dy = g == 0 ? *reinterpret_cast<const bf16x8*>(&dY[16 * w + c][0]) : zero_op();
    // dZ2[s][j] = (sum_o dY[s][o] W3[j][o]) * (H2[s][j] > 0)
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
      const f32x4 acc = mfma16(dy, w3[nt], zero4());
      __bf16 z[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        z[r] = (__bf16)((float)h2[nt][r] > 0.f ? acc[r] : 0.f);
        H2[16 * w + 4 * g + r][16 * nt + c] = z[r];
      }
      store4(&Z2T[16 * nt + c][16 * w + 4 * g], z);
    }
  }
  wave_fence();
  {
    // dZ1[s][i] = (sum_j dZ2[s][j] W2[i][j]) * (H1[s][i] > 0)
    const bf16x8 a0 = lds_op(&H2[16 * w][0]), a1 = lds_op(&H2[16 * w][32]);
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
      f32x4 acc = mfma16(a0, w2[nt][0], zero4());
      acc = mfma16(a1, w2[nt][1], acc);
      __bf16 z[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) z[r] = (__bf16)((float)h1[nt][r] > 0.f ? acc[r] : 0.f);
      store4(&Z1T[16 * nt + c][16 * w + 4 * g], z);
    }
  }
  __syncthreads();
  // ---- weight gradients over the 64 samples, a quarter per wave
  float* part = p.partial + (size_t)blockIdx.x * kMlpParams;
  {
    // dW2[i][j] = sum_s H1^T[i][s] dZ2^T[j][s], rows i = 16 w ..
    const bf16x8 a0 = lds_op(&H1T[16 * w][0]), a1 = lds_op(&H1T[16 * w][32]);
#pragma unroll
    for (int nj = 0; nj < 4; ++nj) {
      f32x4 acc = mfma16(a0, lds_op(&Z2T[16 * nj][0]), zero4());
      acc = mfma16(a1, lds_op(&Z2T[16 * nj][32]), acc);
#pragma unroll
      for (int r = 0; r < 4; ++r) part[kOffW2 + (16 * w + 4 * g + r) * 64 + 16 * nj + c] = acc[r];
    }
    // dW3[j][o] = sum_s H2^T[j][s] dY^T[o][s]
    bf16x8 d0 = zero_op(), d1 = zero_op();
    if (c < 4) {
      d0 = *reinterpret_cast<const bf16x8*>(&dYT[c][8 * g]);
      d1 = *reinterpret_cast<const bf16x8*>(&dYT[c][32 + 8 * g]);
    }
    f32x4 acc = mfma16(lds_op(&H2T[16 * w][0]), d0, zero4());
    acc = mfma16(lds_op(&H2T[16 * w][32]), d1, acc);
    if (c < 4) {
#pragma unroll
      for (int r = 0; r < 4; ++r) part[kOffW3 + (16 * w + 4 * g + r) * 4 + c] = acc[r];
    }
    // dW1[k][i] = sum_s Xh^T[k][s] dZ1^T[i][s], columns i = 16 w ..
    bf16x8 x0 = zero_op(), x1 = zero_op();
    if (c < 5) {
      x0 = *reinterpret_cast<const bf16x8*>(&XhT[c][8 * g]);
      x1 = *reinterpret_cast<const bf16x8*>(&XhT[c][32 + 8 * g]);
    }
    acc = mfma16(x0, lds_op(&Z1T[16 * w][0]), zero4());
    acc = mfma16(x1, lds_op(&Z1T[16 * w][32]), acc);
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (4 * g + r < 5) part[kOffW1 + (4 * g + r) * 64 + 16 * w + c] = acc[r];
  }
  // bias gradients and the loss share, one per wave
  if (w == 0) {
    part[kOffB2 + l] = row_sum(&Z2T[l][0]);
  } else if (w == 1) {
    part[kOffB1 + l] = row_sum(&Z1T[l][0]);
  } else if (w == 2) {
    if (l < 4) part[kOffB3 + l] = row_sum(&dYT[l][0]);
  } else {
    float loss = 0.f;
#pragma unroll
    for (int q = 0; q < 16; ++q) loss += sq[q][l];
    for (int d = 32; d >= 1; d >>= 1) loss += __shfl_xor(loss, d, 64);
    if (l == 0) p.loss_partial[blockIdx.x] = loss;
  }
}

// Sum of the block partials (fixed order: deterministic) -> grad; optionally
// the Adam update of the master weights (lr follows a cosine schedule).
struct AdamParams {
  const float* partial;
  const float* loss_partial;
  int blocks;
  float* master;
  float* m1;
  float* m2;
  TrainWeights* tw;  // bf16 layouts refreshed with each updated parameter
  MlpImage* img;
  int t;             // Adam steps done before this one
  int total_steps;
  float lr;
  float* grad_out;   // may be null
  float* loss_out;   // loss per step of this call, may be null
  int loss_index;    // step index within this call
  int batch;
  int update;
};

// sum + the last `left` <= N partials in order, N loads in flight: those beyond repeat the last
// one, and add the zero that changes no sum.
template <int N>
__device__ __forceinline__ float add_last(const float* at, int left, float sum) {
  float v[N];
#pragma unroll
  for (int q = 0; q < N; ++q) {
    v[q] = *at;
    at += q + 1 < left ? kMlpParams : 0;
  }
#pragma unroll
  for (int q = 0; q < N; ++q) sum += q < left ? v[q] : -0.0f;
  return sum;
}

// One wave per 64 parameters (and one for the loss), so that the 76 waves sit on as many
// CUs. Bound by the latency of the partials, which other XCDs wrote: 64 loads are in flight
// per lane, fewer only where fewer are left, and the additions keep their order. Where each
// load waited for the addition before it, 64 partials took 19.7 us (4.1 now); a step with 63 of
// them 23.5 us where the rest beside groups of 64 was added that way, 10.8 now (64: 10.4).
__global__ __launch_bounds__(64) void k_adam(AdamParams p) {
  constexpr int kFly = 64;
  const int l = threadIdx.x;
  if (blockIdx.x == gridDim.x - 1) {  // loss of this step
    if (!p.loss_out) return;
    float ls = 0.f;
    for (int b0 = 0; b0 < p.blocks; b0 += 64) {
      const float v = b0 + l < p.blocks ? p.loss_partial[b0 + l] : 0.f;
      for (int q = 0; q < min(64, p.blocks - b0); ++q)
        ls += __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v), q));
    }
    if (l == 0) p.loss_out[p.loss_index] = ls / (4.0f * (float)p.batch);
    return;
  }
  const int i = blockIdx.x * 64 + l;
  if (i >= kMlpParams) return;
  const float* part = p.partial + i;
  float m1 = 0.f, m2 = 0.f, w = 0.f;
  if (p.update) {
    m1 = p.m1[i];
    m2 = p.m2[i];
    w = p.master[i];
  }
  float gsum = 0.f;
  int b = 0;
  for (; b + kFly <= p.blocks; b += kFly) {
    float v[kFly];
#pragma unroll
    for (int q = 0; q < kFly; ++q) v[q] = part[(size_t)(b + q) * kMlpParams];
#pragma unroll
    for (int q = 0; q < kFly; ++q) gsum += v[q];
  }
  const int left = p.blocks - b;
  const float* rest = part + (size_t)b * kMlpParams;
  if (left > 32) gsum = add_last<64>(rest, left, gsum);
  else if (left > 16) gsum = add_last<32>(rest, left, gsum);
  else if (left > 8) gsum = add_last<16>(rest, left, gsum);
  else if (left > 2) gsum = add_last<8>(rest, left, gsum);
  else if (left > 0) gsum = add_last<2>(rest, left, gsum);
  if (p.grad_out) p.grad_out[i] = gsum;
  if (p.update) {
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float tt = (float)(p.t + 1);
    const float prog = p.total_steps > 1 ? (float)p.loss_index / (float)(p.total_steps - 1) : 0.f;
    const float lr = p.lr * (0.01f + 0.99f * 0.5f * (1.f + cosf(3.14159265f * fminf(prog, 1.f))));
    const float c1 = 1.f - powf(b1, tt), c2 = 1.f - powf(b2, tt);
    m1 = b1 * m1 + (1.f - b1) * gsum;
    m2 = b2 * m2 + (1.f - b2) * gsum * gsum;
    p.m1[i] = m1;
    p.m2[i] = m2;
    const float mh = m1 / c1;
    const float vh = m2 / c2;
    w = w - lr * mh / (sqrtf(vh) + eps);
    p.master[i] = w;
    scatter_param(i, w, p.tw, p.img);
  }
}

// ---------------------------------------------------------------------------- batch inference

__global__ __launch_bounds__(256) void k_forward(const MlpImage* __restrict__ img, const float* __restrict__ X,
                                                 float* __restrict__ Y, int64_t n) {
  __shared__ __attribute__((aligned(16))) MlpImage s_img;
  __shared__ uint4 s_stage[256];
  {
    const uint4* src = reinterpret_cast<const uint4*>(img);
    uint4* dst = reinterpret_cast<uint4*>(&s_img);
    for (int i = threadIdx.x; i < (int)(sizeof(MlpImage) / 16); i += 256) dst[i] = src[i];
  }
  __syncthreads();
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t jj = j < n ? j : n - 1;  // every lane takes part in the wave-wide product
  float x[kMlpIn], y[kMlpOut];
#pragma unroll
  for (int k = 0; k < kMlpIn; ++k) x[k] = X[5 * jj + k];
  mlp_forward_wave(&s_img, x, y, s_stage + (threadIdx.x & ~63u));
  if (j < n) {
#pragma unroll
    for (int o = 0; o < kMlpOut; ++o) Y[4 * j + o] = y[o];
  }
}

}  // namespace

}  // namespace cphot

// ================================================================================ host API

// Per-block partial gradients and loss shares of cphot_surrogate_gradient_noalloc:
// at most kNoAllocSamples samples, i.e. kNoAllocSamples / 64 blocks, each
// writing all kMlpParams entries of its row and its loss share (so nothing needs
// clearing between calls). 1.23 MB per device, held until the process ends. In host
// code `scratch` only names the symbol: its device address comes from
// hipGetSymbolAddress (once per device, kept in g_scratch_addr).
constexpr int kNoAllocSamples = 4096;
constexpr int kNoAllocBlocks = kNoAllocSamples / 64;
static __device__ __align__(256) float scratch[(size_t)kNoAllocBlocks * cphot::kMlpParams + kNoAllocBlocks];

struct cphot_surrogate {
  cphot_surrogate_desc d;
  int device = 0;
  int max_blocks = 0;
  float* master = nullptr;
  float* m1 = nullptr;
  float* m2 = nullptr;
  float* norm = nullptr;
  float* partial = nullptr;
  float* loss_partial = nullptr;
  int steps_done = 0;  // Adam steps enqueued so far (bias correction)
  double* sums = nullptr;
  cphot::TrainWeights* tw = nullptr;
  cphot::MlpImage* img = nullptr;
  bool normalised = false;
};

namespace {

int sfail(int code, const std::string& m) {
  cphot::set_last_error(m);
  return code;
}

int shfail(hipError_t e, const char* what) { return sfail(CPHOT_ERR_HIP, std::string(what) + ": " + hipGetErrorString(e)); }

// splitmix64 -> uniform in [0, 1): initial weights only
double init_uniform(uint64_t& s) {
  uint64_t z = (s += 0x9E3779B97F4A7C15ull);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z ^= z >> 31;
  return (double)(z >> 11) * (1.0 / 9007199254740992.0);
}

hipError_t pack(cphot_surrogate* s, hipStream_t st) {
  hipLaunchKernelGGL(cphot::k_pack, dim3(16), dim3(256), 0, st, s->master, s->norm, s->tw, s->img);
  return hipGetLastError();
}

// Device address of `scratch` on device `dev` (the current device), looked up on
// the first call per device and kept: each device holds its own copy of the array.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float* g_scratch_addr[kMaxDevices] = {};

int scratch_address(int dev, float** out) {
  if (dev < 0 || dev >= kMaxDevices) return sfail(CPHOT_ERR_INVALID_ARG, "device index beyond 64");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_addr[dev]) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return shfail(e, "hipGetSymbolAddress(scratch)");
    if (!ptr) return sfail(CPHOT_ERR_HIP, "hipGetSymbolAddress(scratch) returned null");
    g_scratch_addr[dev] = static_cast<float*>(ptr);
  }
  *out = g_scratch_addr[dev];
  return CPHOT_OK;
}

}  // namespace

extern "C" {

int cphot_surrogate_create(const cphot_surrogate_desc* desc, cphot_surrogate** out) {
  if (!desc || !out) return sfail(CPHOT_ERR_INVALID_ARG, "null argument");
  *out = nullptr;
  for (int j = 0; j < 5; ++j)
    if (!std::isfinite(desc->in_lo[j]) || !std::isfinite(desc->in_hi[j]) || !(desc->in_hi[j] > desc->in_lo[j]))
      return sfail(CPHOT_ERR_INVALID_ARG, "domain box needs finite lo < hi on every input");
  if (desc->in_lo[1] < 0.0 || desc->in_hi[1] > 1.0)
    return sfail(CPHOT_ERR_INVALID_ARG, "cos(zenith) range must lie in [0, 1]");
  if (desc->max_batch < 64 || desc->max_batch % 64 || desc->max_batch > (1 << 22))
    return sfail(CPHOT_ERR_INVALID_ARG, "max_batch must be a positive multiple of 64 up to 2^22");
  if (desc->geometry != CPHOT_SURROGATE_PLANAR && desc->geometry != CPHOT_SURROGATE_CURVED)
    return sfail(CPHOT_ERR_INVALID_ARG, "unknown surrogate geometry");
  cphot_surrogate* s = new (std::nothrow) cphot_surrogate();
  if (!s) return sfail(CPHOT_ERR_OUT_OF_MEMORY, "host allocation");
  s->d = *desc;
  (void)hipGetDevice(&s->device);
  s->max_blocks = desc->max_batch / 64;
  hipError_t e;
  auto fail_free = [&](hipError_t err, const char* what) {
    cphot_surrogate_destroy(s);
    return err == hipErrorOutOfMemory ? sfail(CPHOT_ERR_OUT_OF_MEMORY, what) : shfail(err, what);
  };
  if ((e = hipMalloc(&s->master, cphot::kMlpParams * 4)) != hipSuccess) return fail_free(e, "hipMalloc");
  if ((e = hipMalloc(&s->m1, cphot::kMlpParams * 4)) != hipSuccess) return fail_free(e, "hipMalloc");
  if ((e = hipMalloc(&s->m2, cphot::kMlpParams * 4)) != hipSuccess) return fail_free(e, "hipMalloc");
  if ((e = hipMalloc(&s->norm, cphot::kMlpNorm * 4)) != hipSuccess) return fail_free(e, "hipMalloc");
  if ((e = hipMalloc(&s->partial, (size_t)s->max_blocks * cphot::kMlpParams * 4)) != hipSuccess)
    return fail_free(e, "hipMalloc");
  if ((e = hipMalloc(&s->loss_partial, (size_t)s->max_blocks * 4)) != hipSuccess) return fail_free(e, "hipMalloc");
  if ((e = hipMalloc(&s->sums, 8 * sizeof(double))) != hipSuccess) return fail_free(e, "hipMalloc");
  if ((e = hipMalloc(&s->tw, sizeof(cphot::TrainWeights))) != hipSuccess) return fail_free(e, "hipMalloc");
  if ((e = hipMalloc(&s->img, sizeof(cphot::MlpImage))) != hipSuccess) return fail_free(e, "hipMalloc");
  // He-uniform initial weights, zero biases
  std::vector<float> w(cphot::kMlpParams, 0.f);
  uint64_t rs = desc->init_seed;
  auto fill = [&](int off, int fan_in, int count) {
    const double lim = std::sqrt(6.0 / fan_in);
    for (int i = 0; i < count; ++i) w[off + i] = (float)((2.0 * init_uniform(rs) - 1.0) * lim);
  };
  fill(cphot::kOffW1, 5, 320);
  fill(cphot::kOffW2, 64, 4096);
  fill(cphot::kOffW3, 64, 256);
  std::vector<float> nrm(cphot::kMlpNorm, 0.f);
  for (int j = 0; j < 5; ++j) {
    nrm[j] = (float)desc->in_lo[j];
    nrm[5 + j] = (float)desc->in_hi[j];
    nrm[10 + j] = (float)(2.0 / (desc->in_hi[j] - desc->in_lo[j]));
  }
  for (int o = 0; o < 4; ++o) nrm[20 + o] = 1.f;
  std::vector<float> zeros(cphot::kMlpParams, 0.f);
  if ((e = hipMemcpy(s->master, w.data(), w.size() * 4, hipMemcpyHostToDevice)) != hipSuccess ||
      (e = hipMemcpy(s->m1, zeros.data(), zeros.size() * 4, hipMemcpyHostToDevice)) != hipSuccess ||
      (e = hipMemcpy(s->m2, zeros.data(), zeros.size() * 4, hipMemcpyHostToDevice)) != hipSuccess ||
      (e = hipMemcpy(s->norm, nrm.data(), nrm.size() * 4, hipMemcpyHostToDevice)) != hipSuccess)
    return fail_free(e, "hipMemcpy");
  if ((e = pack(s, nullptr)) != hipSuccess) return fail_free(e, "pack");
  if ((e = hipDeviceSynchronize()) != hipSuccess) return fail_free(e, "synchronize");
  *out = s;
  return CPHOT_OK;
}

void cphot_surrogate_destroy(cphot_surrogate* s) {
  if (!s) return;
  int prev = 0;
  (void)hipGetDevice(&prev);
  (void)hipSetDevice(s->device);
  for (void* ptr : {(void*)s->master, (void*)s->m1, (void*)s->m2, (void*)s->norm, (void*)s->partial,
                    (void*)s->loss_partial, (void*)s->sums, (void*)s->tw, (void*)s->img})
    if (ptr) (void)hipFree(ptr);
  (void)hipSetDevice(prev);
  delete s;
}

int cphot_surrogate_make_training_set(const cphot_surrogate* s, const cphot_atmosphere* atm, int64_t first,
                                      int64_t n, uint64_t seed, float* X, float* Y, void* stream) {
  if (!s || !atm) return sfail(CPHOT_ERR_INVALID_ARG, "null surrogate or atmosphere");
  if (n < 0 || first < 0) return sfail(CPHOT_ERR_INVALID_ARG, "negative n or first");
  if (n > 0 && (!X || !Y)) return sfail(CPHOT_ERR_INVALID_ARG, "null X or Y");
  cphot::TrainSetParams p;
  std::memset(&p, 0, sizeof(p));
  int rc = cphot::atmosphere_layer_view(atm, &p.layers, &p.lambins, &p.n_layers, &p.n_lam, &p.dh, &p.lam_min,
                                        &p.lam_max);
  if (rc) return sfail(rc, "the surrogate is trained on a layered atmosphere (n_layers > 0)");
  p.moments = cphot::atmosphere_layer_moments(atm);
  if (!p.moments) return sfail(CPHOT_ERR_INVALID_ARG, "the atmosphere has no layer-sum moments");
  const double top = (double)p.dh * p.n_layers;
  if (s->d.in_hi[0] > top || s->d.in_hi[4] > top || s->d.in_lo[4] < 0.0)
    return sfail(CPHOT_ERR_INVALID_ARG, "domain heights must lie inside the layered atmosphere");
  if (s->d.in_lo[3] > p.lam_min || s->d.in_hi[3] < p.lam_max)
    return sfail(CPHOT_ERR_INVALID_ARG, "domain wavelengths must cover the atmosphere's band");
  if (s->d.in_lo[0] < s->d.in_lo[4])
    return sfail(CPHOT_ERR_INVALID_ARG, "domain emission heights must start at or above the lowest observation level");
  {  // the starts are layer boundaries above the observation layer: the box must hold one for every h_obs
    const double dh = (double)p.dh;
    if (!((std::floor(s->d.in_hi[4] / dh) + 1.0) * dh <= s->d.in_hi[0]) ||
        !(std::ceil(s->d.in_lo[0] / dh) * dh <= s->d.in_hi[0]))
      return sfail(CPHOT_ERR_INVALID_ARG, "the emission-height range must hold a layer boundary above every "
                                          "observation layer of the box");
  }
  p.geometry = s->d.geometry;
  p.earth_radius = cphot::atmosphere_earth_radius(atm);
  if (p.geometry == CPHOT_SURROGATE_CURVED && !(p.earth_radius > 1e5 && std::isfinite(p.earth_radius)))
    return sfail(CPHOT_ERR_INVALID_ARG, "a curved surrogate needs the atmosphere's earth_radius");
  if (p.geometry == CPHOT_SURROGATE_CURVED) {
    // every ray of the box must meet the observation sphere on its straight chord (the
    // targets are per metre of that chord): (R + h_e,max) sin(zenith_max) < R + h_obs,min
    const double c = s->d.in_lo[1], sz = std::sqrt(std::max(0.0, (1.0 - c) * (1.0 + c)));
    if (!((p.earth_radius + s->d.in_hi[0]) * sz < p.earth_radius + s->d.in_lo[4]))
      return sfail(CPHOT_ERR_INVALID_ARG, "curved domain box reaches rays that miss the observation sphere: "
                                          "raise the lowest cos zenith or lower the highest emission height");
  }
  if (n == 0) return CPHOT_OK;
  for (int j = 0; j < 5; ++j) {
    p.lo[j] = (float)s->d.in_lo[j];
    p.hi[j] = (float)s->d.in_hi[j];
  }
  p.key0 = (uint32_t)seed;
  p.key1 = (uint32_t)(seed >> 32);
  p.first = first;
  p.n = n;
  p.X = X;
  p.Y = Y;
  const dim3 grid((unsigned)((n + cphot::kSetSamples - 1) / cphot::kSetSamples));
  if (p.geometry == CPHOT_SURROGATE_CURVED)
    hipLaunchKernelGGL(cphot::k_training_set<true>, grid, dim3(cphot::kSetBlock), 0, (hipStream_t)stream, p);
  else
    hipLaunchKernelGGL(cphot::k_training_set<false>, grid, dim3(cphot::kSetBlock), 0, (hipStream_t)stream, p);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? CPHOT_OK : shfail(e, "launch training set");
}

int cphot_surrogate_fit_normalization(cphot_surrogate* s, const float* Y, int64_t n, void* stream) {
  if (!s || !Y || n < 2) return sfail(CPHOT_ERR_INVALID_ARG, "need a surrogate and at least two targets");
  hipStream_t st = (hipStream_t)stream;
  hipLaunchKernelGGL(cphot::k_zero_f64, dim3(1), dim3(64), 0, st, s->sums, 8);
  const int blocks = (int)std::min<int64_t>((n + 255) / 256, 1024);
  hipLaunchKernelGGL(cphot::k_output_sums, dim3(blocks), dim3(256), 0, st, Y, n, s->sums);
  hipLaunchKernelGGL(cphot::k_output_norm, dim3(1), dim3(64), 0, st, (const double*)s->sums, n, s->norm);
  hipError_t e = pack(s, st);
  if (e != hipSuccess) return shfail(e, "normalisation");
  s->normalised = true;
  return CPHOT_OK;
}

static int run_steps(cphot_surrogate* s, const float* X, const float* Y, int64_t n, int batch, int steps,
                     int total_steps, float lr, int64_t start, float* loss_out, float* grad_out, int update,
                     float* partial, float* loss_partial, hipStream_t st) {
  const int blocks = batch / 64;
  for (int k = 0; k < steps; ++k) {
    cphot::StepParams sp;
    sp.X = X;
    sp.Y = Y;
    sp.n = n;
    sp.start = (start + (int64_t)k * batch) % n;
    sp.batch = batch;
    sp.norm = s->norm;
    sp.master = s->master;
    sp.tw = s->tw;
    sp.partial = partial;
    sp.loss_partial = loss_partial;
    hipLaunchKernelGGL(cphot::k_train_step, dim3(blocks), dim3(256), 0, st, sp);
    cphot::AdamParams ap;
    ap.partial = partial;
    ap.loss_partial = loss_partial;
    ap.blocks = blocks;
    ap.master = s->master;
    ap.m1 = s->m1;
    ap.m2 = s->m2;
    ap.tw = s->tw;
    ap.img = s->img;
    ap.t = s->steps_done;
    ap.total_steps = total_steps;
    ap.lr = lr;
    ap.grad_out = grad_out;
    ap.loss_out = loss_out;
    ap.loss_index = k;
    ap.batch = batch;
    ap.update = update;
    hipLaunchKernelGGL(cphot::k_adam, dim3((cphot::kMlpParams + 63) / 64 + 1), dim3(64), 0, st, ap);
    if (update) ++s->steps_done;
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return shfail(e, "training step");
  }
  return CPHOT_OK;
}

int cphot_surrogate_train(cphot_surrogate* s, const float* X, const float* Y, int64_t n, int32_t batch,
                          int32_t steps, float lr, float* loss_out, void* stream) {
  if (!s || !X || !Y) return sfail(CPHOT_ERR_INVALID_ARG, "null argument");
  if (!s->normalised) return sfail(CPHOT_ERR_UNSUPPORTED, "fit the output normalisation first");
  if (batch < 64 || batch % 64 || batch > s->d.max_batch)
    return sfail(CPHOT_ERR_INVALID_ARG, "batch must be a multiple of 64 up to max_batch");
  if (n < batch) return sfail(CPHOT_ERR_INVALID_ARG, "training set smaller than one batch");
  if (steps < 0 || !(lr > 0.f) || !std::isfinite(lr)) return sfail(CPHOT_ERR_INVALID_ARG, "bad steps or lr");
  return run_steps(s, X, Y, n, batch, steps, steps, lr, 0, loss_out, nullptr, 1, s->partial, s->loss_partial,
                   (hipStream_t)stream);
}

int cphot_surrogate_gradient(cphot_surrogate* s, const float* X, const float* Y, int64_t n, float* grad,
                             float* loss, void* stream) {
  if (!s || !X || !Y || !grad) return sfail(CPHOT_ERR_INVALID_ARG, "null argument");
  if (n < 64 || n % 64 || n > s->d.max_batch)
    return sfail(CPHOT_ERR_INVALID_ARG, "n must be a multiple of 64 up to max_batch");
  return run_steps(s, X, Y, n, (int)n, 1, 1, 1.f, 0, loss, grad, 0, s->partial, s->loss_partial,
                   (hipStream_t)stream);
}

int cphot_surrogate_gradient_noalloc(cphot_surrogate* s, const float* X, const float* Y, int64_t n, float* grad,
                                     float* loss, void* stream) {
  if (!s || !X || !Y || !grad) return sfail(CPHOT_ERR_INVALID_ARG, "null argument");
  if (n < 64 || n % 64 || n > kNoAllocSamples)
    return sfail(CPHOT_ERR_INVALID_ARG, "n must be a multiple of 64 up to 4096 (the static workspace)");
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return shfail(e, "hipGetDevice");
  if (dev != s->device) return sfail(CPHOT_ERR_INVALID_ARG, "call on the device the surrogate was created on");
  float* ws = nullptr;
  const int rc = scratch_address(dev, &ws);
  if (rc) return rc;
  return run_steps(s, X, Y, n, (int)n, 1, 1, 1.f, 0, loss, grad, 0, ws, ws + (size_t)kNoAllocBlocks * cphot::kMlpParams,
                   (hipStream_t)stream);
}

int cphot_surrogate_forward(const cphot_surrogate* s, const float* X, float* Y, int64_t n, void* stream) {
  if (!s) return sfail(CPHOT_ERR_INVALID_ARG, "null surrogate");
  if (n < 0 || (n > 0 && (!X || !Y))) return sfail(CPHOT_ERR_INVALID_ARG, "bad buffers");
  if (n == 0) return CPHOT_OK;
  hipLaunchKernelGGL(cphot::k_forward, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                     (const cphot::MlpImage*)s->img, X, Y, n);
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? CPHOT_OK : shfail(e, "launch forward");
}

int cphot_surrogate_get_params(const cphot_surrogate* s, float* params, float* norm) {
  if (!s) return sfail(CPHOT_ERR_INVALID_ARG, "null surrogate");
  hipError_t e = hipDeviceSynchronize();
  if (e == hipSuccess && params) e = hipMemcpy(params, s->master, cphot::kMlpParams * 4, hipMemcpyDeviceToHost);
  if (e == hipSuccess && norm) e = hipMemcpy(norm, s->norm, cphot::kMlpNorm * 4, hipMemcpyDeviceToHost);
  return e == hipSuccess ? CPHOT_OK : shfail(e, "get params");
}

int cphot_surrogate_set_params(cphot_surrogate* s, const float* params, const float* norm) {
  if (!s) return sfail(CPHOT_ERR_INVALID_ARG, "null surrogate");
  hipError_t e = hipDeviceSynchronize();
  if (e == hipSuccess && params) e = hipMemcpy(s->master, params, cphot::kMlpParams * 4, hipMemcpyHostToDevice);
  if (e == hipSuccess && norm) {
    e = hipMemcpy(s->norm, norm, cphot::kMlpNorm * 4, hipMemcpyHostToDevice);
    s->normalised = true;
  }
  if (e == hipSuccess) e = pack(s, nullptr);
  if (e == hipSuccess) e = hipDeviceSynchronize();
  return e == hipSuccess ? CPHOT_OK : shfail(e, "set params");
}

}  // extern "C"

namespace cphot {
const MlpImage* surrogate_image(const cphot_surrogate* s) { return s ? s->img : nullptr; }
bool surrogate_ready(const cphot_surrogate* s) { return s && s->normalised; }
int surrogate_geometry(const cphot_surrogate* s) { return s ? s->d.geometry : CPHOT_SURROGATE_PLANAR; }
}  // namespace cphot
