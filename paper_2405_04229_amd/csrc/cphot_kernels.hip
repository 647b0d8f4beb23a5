// Photon generation and propagation kernels for gfx950.
//
// One kernel per (block size, transport, detector, mode). A wave works on its own
// tile of 64 consecutive segments, with no block barrier in the loop over tiles:
//   1. coalesced SoA load, one segment per lane; FP64 yield and the stochastically
//      rounded record count (Sec. 2.2.1); FP32 per-segment state (cone angle,
//      rotation bisector, start point, first Philox rounds) into the wave's LDS
//      slots, sorted by start layer under refracting transports;
//   2. wave scans of the counts -> flat record numbers, Cherenkov records first,
//      then fluorescence, each kind in rounds of 64;
//   3. a round is one record per lane: its slot from a push of the slot starts and
//      a running maximum over the lanes, then the record's Philox block, the photon
//      on the cone (Sec. 4.2), its transport (Sec. 3.4.1 straight / Sec. 3.4.2
//      layered), absorption (Sec. 2.3.2) and its bin (LDS-privatised histogram or
//      global atomics); upward photons leave first (Sec. 5.3.4).
// Photons live in registers only; nothing per photon touches HBM except the
// final bin increment. The waves of a block share the LDS histogram and the tables.
#include "cphot_device.h"
#include "cphot_internal.h"
#include "cphot_mlp.h"

#include <algorithm>
#include <type_traits>

namespace cphot {

namespace {

struct SegResult {
  int32_t n;       // Cherenkov records
  int32_t status;  // 0 ok, 1 below the Cherenkov threshold, 2 skipped
  float cos_t, sin_t, a0, a1, a2;
  double mu;       // expected Cherenkov records
  int32_t nf[3];   // fluorescence records per band
  float inv_q;     // 1 / pre-emission reduction factor (1 without reduction)
  // DISPERSIVE: g(lambda) = beta n(lambda, h_mid) - 1 = disp_gm + disp_a (R(lambda) - R(lam_min))
  float disp_a, disp_gm;
};

// Per-segment yield in FP64 with IEEE basic operations only and no
// contraction, in the fixed order that makes the record count reproducible
// bit for bit on any IEEE machine. EXT: Poisson counts and the dispersive
// spectrum are compiled in (kernels without them never see those settings).
template <bool EXT>
__device__ __forceinline__ SegResult segment_setup(const KParams& p, float fx0, float fy0, float fz0, float fx1,
                                                float fy1, float fz1, float fbeta, float fq, float fdedx,
                                                uint64_t id) {
#pragma clang fp contract(off)
  SegResult r{0, 0, 0.f, 0.f, 0.f, 0.f, 0.f, 0.0, {0, 0, 0}, 1.f};
  const bool cher = (p.emission & CPHOT_EMIT_CHERENKOV) != 0;
  const bool fluor = (p.emission & CPHOT_EMIT_FLUORESCENCE) != 0;
  if (!__builtin_isfinite(fx0) || !__builtin_isfinite(fy0) || !__builtin_isfinite(fz0) ||
      !__builtin_isfinite(fx1) || !__builtin_isfinite(fy1) || !__builtin_isfinite(fz1) ||
      !__builtin_isfinite(fbeta) || !__builtin_isfinite(fq) || (fluor && !__builtin_isfinite(fdedx))) {
    r.status = 2;
    return r;
  }
  const double beta = (double)fbeta;
  if (!(beta > 0.0 && beta < 1.0)) {
    r.status = 2;
    return r;
  }
  const double dx = (double)fx1 - (double)fx0, dy = (double)fy1 - (double)fy0, dz = (double)fz1 - (double)fz0;
  const double L = sqrt(dx * dx + dy * dy + dz * dz);
  if (!(L > 0.0)) {
    r.status = 2;
    return r;
  }
  // pre-emission reduction (Sec. 4.3.1): the bound q of the layer holding the
  // segment's lowest point scales every expected count before rounding
  double q = 1.0;
  if (p.red) {
    const double hmin = (double)fz0 < (double)fz1 ? (double)fz0 : (double)fz1;
    double x = hmin / p.dh64;
    if (x < 0.0) x = 0.0;
    int64_t li = (int64_t)floor(x);
    if (li > p.n_layers - 1) li = p.n_layers - 1;
    q = p.red[li];
    r.inv_q = q > 0.0 ? (float)(1.0 / q) : 0.f;
  }
  // one Philox block per segment: word 0 rounds the Cherenkov yield, words 1..3
  // the fluorescence bands
  const uint4 w = philox(0u, (uint32_t)id, (uint32_t)(id >> 32), TAG_SEGMENT, p.key0, p.key1);
  if (cher) {
    // refractivity at the midpoint: direct index mapping into the FP64 table and
    // linear interpolation (Sec. 4.1), heights clamped to the table
    const double hm = 0.5 * ((double)fz0 + (double)fz1);
    double x = hm / p.step;
    if (x < 0.0) x = 0.0;
    if (x > (double)p.n_tab) x = (double)p.n_tab;
    double fi = floor(x);
    int64_t idx = (int64_t)fi;
    if (idx > p.n_tab - 1) {
      idx = p.n_tab - 1;
      fi = (double)idx;
    }
    const double frac = x - fi;
    double delta = (1.0 - frac) * p.tab[idx] + frac * p.tab[idx + 1];
    const double eps = 1.0 - beta;
    if (EXT && p.spectrum == CPHOT_SPECTRUM_DISPERSIVE) {
      // records are drawn for the largest cone, n at lam_min; each record's own
      // angle follows from its wavelength
      r.disp_a = (float)(delta * (1.0 - eps) * p.disp_inv_rref);
      delta = delta * p.disp_dmax;
    }
    // threshold beta n > 1 through g = beta n - 1 = delta - eps - eps delta, eps = 1 - beta
    const double g = delta - eps - eps * delta;
    if (!(g > 0.0)) {
      r.status = 1;
    } else {
      const double s2 = g * (g + 2.0) / ((1.0 + g) * (1.0 + g));
      r.disp_gm = (float)g;
      const double z2 = (double)fq * (double)fq;
      double mu = p.K * z2;
      mu = mu * L;
      mu = mu * s2;
      mu = mu / (double)p.bunch;
      if (!(mu < (double)(1 << kMaxRecordsPerSegmentLog2))) {
        r.status = 2;
        return r;
      }
      mu = mu * q;
      r.mu = mu;
      if (EXT && p.poisson) {
        const int64_t n = poisson_count(mu, w.x, id, TAG_POISSON, p.key0, p.key1);
        if (n >= (int64_t(1) << kMaxRecordsPerSegmentLog2)) {
          r.status = 2;
          r.n = 0;
          return r;
        }
        r.n = (int32_t)n;
      } else {
        const double fl = floor(mu);
        const double u = (double)w.x * (1.0 / 4294967296.0);
        r.n = (int32_t)fl + (u < mu - fl ? 1 : 0);
      }
      r.cos_t = (float)(1.0 / (1.0 + g));
      r.sin_t = (float)sqrt(s2);
    }
  }
  if (fluor && fdedx > 0.0f) {
    // per band: Y_b dE/dx L / 2 (lower hemisphere only)
    const uint32_t wb[3] = {w.y, w.z, w.w};
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      double mu = p.fl_yield[b] * (double)fdedx;
      mu = mu * L;
      mu = mu * 0.5;
      mu = mu / (double)p.bunch;
      if (!(mu < (double)(1 << kMaxRecordsPerSegmentLog2))) {
        SegResult bad{0, 2, 0.f, 0.f, 0.f, 0.f, 0.f, 0.0, {0, 0, 0}, 1.f};
        return bad;
      }
      mu = mu * q;
      if (EXT && p.poisson) {
        const int64_t n = poisson_count(mu, wb[b], id, TAG_POISSON + 1 + b, p.key0, p.key1);
        if (n >= (int64_t(1) << kMaxRecordsPerSegmentLog2)) {
          SegResult bad{0, 2, 0.f, 0.f, 0.f, 0.f, 0.f, 0.0, {0, 0, 0}, 1.f};
          return bad;
        }
        r.nf[b] = (int32_t)n;
      } else {
        const double fl = floor(mu);
        const double u = (double)wb[b] * (1.0 / 4294967296.0);
        r.nf[b] = (int32_t)fl + (u < mu - fl ? 1 : 0);
      }
    }
  }
  // bisector of the cone axis (0,0,-1) and the track direction; the rotation
  // is M = 2 a a^T - I (Euler-Rodrigues, 180 degrees, Sec. 4.2)
  const double P0 = dx / L, P1 = dy / L, P2 = dz / L;
  if (1.0 - P2 < 1e-6) {
    r.a0 = 1.f;  // 2 a a^T - I with a = x-hat: a half turn about x
  } else {
    const double b2 = P2 - 1.0;
    const double na = sqrt(P0 * P0 + P1 * P1 + b2 * b2);
    r.a0 = (float)(P0 / na);
    r.a1 = (float)(P1 / na);
    r.a2 = (float)(b2 / na);
  }
  return r;
}

// Per-block copy in LDS of the small kernel-argument arrays that records index
// per lane (Linsley pieces, fluorescence band wavelengths): indexing argument
// memory per lane would become vector loads from it, and holding the values in
// scalar registers would add to a scalar register file that is already full.
struct KConst {
  float4 lin[5];  // (lower bound (m), a, b, 1/c (1/cm)) per Linsley piece
  float4 fl;      // band wavelengths (nm)
  // hardware reciprocals of launch constants (curved shells): 1 / r_obs, 1 / R^2,
  // 1 / (b_{obs+1} r_obs)
  float4 rc;
};

__device__ __forceinline__ void load_kconst(const KParams& p, KConst& k, int tid) {
  if (tid == 6) k.rc = make_float4(rcp_fast(p.r_obs), rcp_fast(p.Rf * p.Rf), rcp_fast((p.Rf + p.h_obs1) * p.r_obs), 0.f);
  if (tid < 5) k.lin[tid] = make_float4(p.hb[tid], p.la[tid], p.lb[tid], p.linv_c[tid]);
  if (tid == 5) k.fl = make_float4(p.fl_lambda[0], p.fl_lambda[1], p.fl_lambda[2], 0.f);
}

// Linsley vertical depth in FP32 (g/cm^2).
__device__ __forceinline__ float depth_f(const KConst& k, float h) {
  int i = 0;
#pragma unroll
  for (int j = 1; j < 5; ++j) i += (h >= k.lin[j].x) ? 1 : 0;
  const float4 c = k.lin[i];
  const float hcm = h * 100.0f;
  if (i < 4) return c.y + c.z * __expf(-hcm * c.w);
  return c.y - c.z * hcm * c.w;
}

// Squared horizontal distance from (qx, qy) on the observation level to the
// nearest sphere centre of the shower's array (indices clamped to the array).
__device__ __forceinline__ float nearest_sphere_d2(const KParams& p, float core_x, float core_y, float qx, float qy) {
  const float cx0 = core_x - p.half_x, cy0 = core_y - p.half_y;
  const float fi = fminf(fmaxf(rintf((qx - cx0) * p.inv_pitch), 0.f), (float)(p.snx - 1));
  const float fj = fminf(fmaxf(rintf((qy - cy0) * p.inv_pitch), 0.f), (float)(p.sny - 1));
  const float ex = qx - fmaf(fi, p.pitch, cx0), ey = qy - fmaf(fj, p.pitch, cy0);
  return fmaf(ex, ex, ey * ey);
}

// Data-reduction bounds (filter levels 1 and 3, Sec. 4.3.2 / 4.3.4), conservative:
// a photon reaching a sphere of radius r crosses the observation level within
// r / cos(final zenith) of its centre, and its crossing lies within the
// refraction bound of its straight line's: H tan(z) E (1 + 3 tan^2 z) x 1.1 + 0.5 m,
// E the largest |n_i - n_j| / n_i above the observation layer (|tan z_i - tan z| <=
// tan z (E + 0.77 x) with x = 2.2 tan^2 z E <= 0.25). Directions steeper than
// cos z = 0.2, or with x > 0.25, are never cut. `slack` covers FP32 rounding.
__device__ __forceinline__ float cut_slack(float qx, float qy, float core_x, float core_y, float H) {
  return 0.5f + 1e-5f * (fabsf(qx - core_x) + fabsf(qy - core_y) + H);
}

// Filter level 1: can any photon of this segment's Cherenkov cone (half-angle
// theta, from any point of the segment) reach a sphere? The cone's straight lines
// land within H theta / cos^2(zeta + theta) of the axis's landing point (the
// gnomonic projection stretches arcs by at most sec^2 of the largest zenith
// angle), the same point for every point of the segment.
__device__ __forceinline__ bool track_may_hit(const KParams& p, float x0, float y0, float z0, float x1, float y1,
                                              float z1, float cos_t, float sin_t, float core_x, float core_y) {
  const float dx = x1 - x0, dy = y1 - y0, dz = z1 - z0;
  const float L = sqrt_fast(fmaf(dx, dx, fmaf(dy, dy, dz * dz)));
  if (!(L > 0.f)) return true;
  const float iL = rcp_fast(L);
  const float cz = -dz * iL, sz = sqrt_fast(fmaxf((1.0f - cz) * (1.0f + cz), 0.f));
  const float cmin = fmaf(cz, cos_t, -sz * sin_t);  // cos of the steepest cone direction
  if (!(cmin > 0.2f)) return true;
  const float H = fmaxf(z0, z1) - p.h_obs;
  if (!(H > 0.f)) return true;
  const float ic = rcp_fast(cmin);
  const float t2 = (1.0f - cmin * cmin) * ic * ic, tmax = sqrt_fast(t2);
  const float x = 2.2f * t2 * p.cut_e;
  if (!(x <= 0.25f)) return true;
  const float Rfp = H * (1.01f * sin_t) * ic * ic;
  const float dref = fmaf(H * tmax * p.cut_e * fmaf(3.0f, t2, 1.0f), 1.1f, 0.5f);
  const float reff = p.radius * ic * rcp_fast(sqrt_fast(1.0f - x));
  const float s = (p.h_obs - z0) * rcp_fast(dz);  // in units of the segment vector from its start
  const float qx = fmaf(s, dx, x0), qy = fmaf(s, dy, y0);
  const float lim = Rfp + dref + reff + cut_slack(qx, qy, core_x, core_y, H);
  return nearest_sphere_d2(p, core_x, core_y, qx, qy) <= lim * lim;
}

// Filter level 3: can this photon, emitted at height Pz > h_obs going down, reach
// a sphere? Its straight line's crossing of the observation level against the
// nearest sphere centre.
__device__ __forceinline__ bool photon_may_hit(const KParams& p, float Px, float Py, float Pz, float ux, float uy,
                                               float uz, float core_x, float core_y) {
  const float c = -uz;
  if (!(c > 0.2f)) return true;
  const float H = Pz - p.h_obs;
  const float ic = rcp_fast(c);
  const float t2 = fmaf(ux, ux, uy * uy) * ic * ic;
  const float x = 2.2f * t2 * p.cut_e;
  if (!(x <= 0.25f)) return true;
  const float dref = fmaf(H * sqrt_fast(t2) * p.cut_e * fmaf(3.0f, t2, 1.0f), 1.1f, 0.5f);
  const float reff = p.radius * ic * rcp_fast(sqrt_fast(1.0f - x));
  const float s = H * ic;
  const float qx = fmaf(s, ux, Px), qy = fmaf(s, uy, Py);
  const float lim = reff + dref + cut_slack(qx, qy, core_x, core_y, H);
  return nearest_sphere_d2(p, core_x, core_y, qx, qy) <= lim * lim;
}

// Distance from (qx, qy) on the observation level to the shower's ground grid
// (zero inside it), squared.
__device__ __forceinline__ float grid_out_d2(const KParams& p, float core_x, float core_y, float qx, float qy) {
  const float gx0 = core_x - p.half_x, gy0 = core_y - p.half_y;
  const float gx1 = fmaf((float)p.nx, p.cell, gx0), gy1 = fmaf((float)p.ny, p.cell, gy0);
  const float dx = fmaxf(fmaxf(gx0 - qx, qx - gx1), 0.f), dy = fmaxf(fmaxf(gy0 - qy, qy - gy1), 0.f);
  return fmaf(dx, dx, dy * dy);
}

// Filter level 3 for the ground grid over planar layers: the photon's straight
// line against the grid rectangle, widened by the refraction bound of the sphere
// cut (the landing point moves by at most H tan(z) E (1 + 3 tan^2 z) x 1.1 + 0.5 m).
__device__ __forceinline__ bool grid_may_hit(const KParams& p, float Px, float Py, float Pz, float ux, float uy,
                                             float uz, float core_x, float core_y) {
  const float c = -uz;
  if (!(c > 0.2f)) return true;
  const float H = Pz - p.h_obs;
  const float ic = rcp_fast(c);
  const float t2 = fmaf(ux, ux, uy * uy) * ic * ic;
  if (!(2.2f * t2 * p.cut_e <= 0.25f)) return true;
  const float dref = fmaf(H * sqrt_fast(t2) * p.cut_e * fmaf(3.0f, t2, 1.0f), 1.1f, 0.5f);
  const float s = H * ic;
  const float qx = fmaf(s, ux, Px), qy = fmaf(s, uy, Py);
  const float lim = dref + cut_slack(qx, qy, core_x, core_y, H);
  return grid_out_d2(p, core_x, core_y, qx, qy) <= lim * lim;
}

// Filter level 3 for the ground grid over spherical shells, an exact bound. With the
// refractive index non-decreasing downwards, Bouguer's invariant n r sin(z) gives
// sin z <= sin z_s at every radius (z_s of the straight line from the same start), so
// the ray reaches the sphere R + h_obs whenever the straight line does, never turns,
// and tan z_s - tan z <= E tan z_s sec^2 z_s with E >= (n(r) - n_start) / n(r). The
// central angle swept falls short of the straight line's psi_s by at most
// E sec^2(z_end) psi_s (z_end the straight line's local zenith at the sphere, its
// largest), and the vertical projection onto the ground plane does not stretch arcs:
// the arrival lies within E sec^2(z_end) (R + h_obs) psi_s of the straight line's.
// Rays whose straight line misses the sphere are never cut.
__device__ __forceinline__ bool curved_may_land(const KParams& p, float Px, float Py, float Pz, float ux,
                                                float uy, float uz, float rq, float h0, float core_x,
                                                float core_y) {
  const float Rf = p.Rf, r1 = p.r_obs;
  const float irq = rcp_fast(rq);
  const float c0 = -fmaf(ux, Px * irq, fmaf(uy, Py * irq, uz * ((Pz + Rf) * irq)));
  if (!(c0 > 0.f)) return true;
  const float drs = (h0 - p.h_obs) * (rq + r1);  // r0^2 - r1^2
  const float rc = rq * c0;
  const float disc = fmaf(rc, rc, -drs);
  if (!(disc > 0.f)) return true;
  const float s_ch = drs * rcp_fast(rc + sqrt_fast(disc));
  const float s0 = sqrt_fast(fmaxf((1.0f - c0) * (1.0f + c0), 0.f));
  const float se = fminf(rq * s0 * rcp_fast(r1), 1.0f);  // sin z_end
  const float sec2 = rcp_fast(fmaxf((1.0f - se) * (1.0f + se), 1e-30f));
  const float psi_s = asinf(fminf(s_ch * s0 * rcp_fast(r1), 1.0f));
  const float qx = fmaf(s_ch, ux, Px), qy = fmaf(s_ch, uy, Py);
  const float lim = fmaf(p.cut_e * sec2, r1 * psi_s * 1.1f, 1.0f) + 1e-5f * (fabsf(qx - core_x) + fabsf(qy - core_y) + s_ch);
  return grid_out_d2(p, core_x, core_y, qx, qy) <= lim * lim;
}

// Integral of n - 1 from height lo to height hi (m), closed form per profile.
__device__ __forceinline__ float opt_integral(const KParams& p, float lo, float hi, float X_lo, float X_hi) {
  if (p.profile == CPHOT_PROFILE_LINSLEY5) return p.opt_scale * (X_lo - X_hi);
  if (p.profile == CPHOT_PROFILE_HOMOGENEOUS) return p.opt_scale * (hi - lo);
  const float t = p.h_top;
  const float a = fminf(fmaxf(lo, 0.f), t), b = fminf(fmaxf(hi, 0.f), t);
  return p.opt_scale * ((b - a) - (b * b - a * a) / (2.f * t));
}

// Survival threshold of a record, times 2^24 (the records' uniforms stay 24-bit
// integers in FP32; scaling both sides by a power of two changes no decision):
// exp(-tau), times the detector efficiency of its wavelength bin and divided by its
// segment's reduction factor when set (the detection probability over the probability
// the record was generated with). Without efficiency the table holds 2^24, without
// reduction 1/q is 1: no branches. Under the dispersive spectrum the uniform compared
// with it is u / p_emit.
__device__ __forceinline__ float survival_threshold(const float* __restrict__ s_eff, float tau, int kb,
                                                    float inv_q) {
  return __expf(-tau) * (s_eff[kb] * inv_q);
}

// A launch constant kept in a register across the record loop, in the kernels with
// registers to spare (kept: 1 scalar, 2 vector for floats). The statement is empty but
// opaque: without it the register allocator reads the value again from the argument
// memory in every round, a scalar load and a wait each (ten a round in the telescope
// kernel, which gains 3 %; batched straight rays 6 %, the network 1.5 %). The curved
// kernels' scalar registers overflow with it and the lane reads cost more than the loads
// (inclined 14.9 against 14.5 ms): 0.
template <int KEPT>
__device__ __forceinline__ float hold(float v) {
  if constexpr (KEPT == 2) asm("" : "+v"(v));
  if constexpr (KEPT == 1) asm("" : "+s"(v));
  return v;
}
template <int KEPT, class T>
__device__ __forceinline__ T hold(T v) {
  if constexpr (KEPT != 0) asm("" : "+s"(v));
  return v;
}

// The kernel arguments that every record reads (fields as in KParams; each instance keeps
// those it uses). The others are read where they are used (fresh_params).
template <int KEPT>
struct Hot {
  uint32_t key0, key1;
  int32_t spectrum, cuts, n_lam, n_layers, obs_layer;
  float lam_min, inv_lam_min, inv_lam_span24, lam_scale, h_obs, dh, inv_dh;
  float series_tmax;
  const float4* moments;
  int32_t nx, ny, snx, sny, n_t;
  float inv_cell, pitch, inv_pitch, radius, inv_dt;
  float Rf, two_Rf, r_obs, h_obs1, d_obs1, two_Rf_dh, inv_dh_walk, shell_rho, shell_tmax;
  const float* shells;
  double nx64, ny64, inv_cell64;
  int32_t hist_tw;

  __device__ __forceinline__ explicit Hot(const KParams& p) {
#define CPHOT_HOT(f) f = hold<KEPT>(p.f);
    CPHOT_HOT(key0) CPHOT_HOT(key1) CPHOT_HOT(spectrum) CPHOT_HOT(cuts) CPHOT_HOT(n_lam) CPHOT_HOT(n_layers)
    CPHOT_HOT(obs_layer) CPHOT_HOT(lam_min) CPHOT_HOT(inv_lam_min) CPHOT_HOT(inv_lam_span24) CPHOT_HOT(lam_scale)
    CPHOT_HOT(h_obs) CPHOT_HOT(dh) CPHOT_HOT(inv_dh) CPHOT_HOT(series_tmax) CPHOT_HOT(moments) CPHOT_HOT(nx)
    CPHOT_HOT(ny) CPHOT_HOT(snx) CPHOT_HOT(sny) CPHOT_HOT(n_t) CPHOT_HOT(inv_cell) CPHOT_HOT(pitch)
    CPHOT_HOT(inv_pitch) CPHOT_HOT(radius) CPHOT_HOT(inv_dt) CPHOT_HOT(Rf) CPHOT_HOT(two_Rf) CPHOT_HOT(r_obs)
    CPHOT_HOT(h_obs1) CPHOT_HOT(d_obs1) CPHOT_HOT(two_Rf_dh) CPHOT_HOT(inv_dh_walk) CPHOT_HOT(shell_rho)
    CPHOT_HOT(shell_tmax) CPHOT_HOT(shells) CPHOT_HOT(nx64) CPHOT_HOT(ny64) CPHOT_HOT(inv_cell64) CPHOT_HOT(hist_tw)
#undef CPHOT_HOT
  }
};

template <int T>
constexpr bool kMlpTransport = (T == CPHOT_TRANSPORT_SURROGATE || T == kTransportCurvedSurrogate);

// Record states, times 8: a record adds 1 << state to its lane's packed counts.
constexpr uint32_t kStateUp = 8, kStateAbsorbed = 16, kStateOutside = 24, kStateNotEmitted = 32;
// A record that the fast path does not serve: its transport is redone by the
// exact tracer in a separate pass over compacted records.
constexpr uint32_t kStateDeferred = 56;

struct Photon {
  uint32_t state;
  int32_t bin, tbin, culled;
  int32_t ix, iy;  // grid cell
  float x, y, z, t, tau, lam, u3, ux, uy, uz;
};

// LDS of a block that every record reads.
struct Tables {
  const float4* lay;
  const float2* lam;
  const MlpImage* img;
  const KConst* k;
  const float* eff;   // detector efficiency per wavelength bin, times 2^24
  uint4* stage;       // this wave's staging of the network's inputs and outputs
};

// Per-segment state of a record, read from the wave's slot: q0 = start point,
// cos(theta); q1 = (end - start) 2^-24, sin(theta) (DISPERSIVE: the terms of
// beta n(lambda) - 1 in place of the angle); q2 = rotation bisector, depth at the
// start (straight rays) or 1 / q; q3 = Philox words of the segment's id
// (philox_segment), fluorescence records of band 0 (bit pattern); fl01 = fluorescence
// records of bands 0 and 1; straight rays: depth change 2^-24 and 1 / q on their own.
struct SegState {
  float4 q0, q1, q2, q3;
  uint32_t fl01;
  float dX, inv_q;
};

// The shower that the wave's records belong to: the same in every lane.
struct ShowerState {
  int sh;
  float core_x, core_y, axx, axy, axz;
  float x0, y0;      // first cell's edge (GRID) or first sphere's centre (SPHERES)
  double x64, y64;   // first cell's edge in FP64 (curved arrival points)
};

// One record: emission, transport, absorption, detection. `fl`: fluorescence record,
// `kk` its index among the segment's records of its kind. With the surrogate
// transport every lane of the wave must call this together (`valid` marks the
// lanes that carry a real record); the network is evaluated before any lane
// leaves. H: the arguments of the common path (Hot, or KParams where few records go).
// ROWS: list mode, where every record's arrival time is written, not only a binned one's.
template <int TRANSPORT, int DETECTOR, bool NEED_TIME, bool ROWS, bool EXT, class K>
__device__ __forceinline__ void trace(const K& H, const KParams& p, const Tables& T, const SegState& g,
                                      const ShowerState& S, bool fl, uint32_t kk, bool valid, Photon& o) {
  const float4* s_lay = T.lay;
  const float2* s_lam = T.lam;
  const MlpImage* s_img = T.img;
  const KConst* s_k = T.k;
  const float* s_eff = T.eff;
  uint4* s_stage = T.stage;
  const float core_x = S.core_x, core_y = S.core_y, axx = S.axx, axy = S.axy, axz = S.axz;
  float f, lam, u3, ux, uy, uz;  // f and u3 as 24-bit integers
  bool emitted = true;
  float inv_pe = 1.f;
  if (!fl) {
    const uint4 w = philox_record(g.q3, kk, TAG_CHERENKOV, H.key0, H.key1);
    f = (float)(w.x >> 8);
    float sphi, cphi;
    // the cone azimuth needs sin and cos only to about 2e-5: its error enters the
    // direction times sin(theta) < 0.025; the hardware sine takes revolutions
    const float ua = u24(w.y);
    sphi = __builtin_amdgcn_sinf(ua);
    cphi = __builtin_amdgcn_cosf(ua);
    const float u2 = (float)(w.z >> 8);
    lam = (H.spectrum == CPHOT_SPECTRUM_UNIFORM) ? H.lam_min + p.lam_span24 * u2
                                                 : rcp_fast(H.inv_lam_min - u2 * H.inv_lam_span24);
    u3 = (float)(w.w >> 8);
    float cos_t = g.q0.w, sin_t = g.q1.w;
    if (EXT && H.spectrum == CPHOT_SPECTRUM_DISPERSIVE) {
      // angle of this wavelength (Eq. 2.5) and the record's emission probability
      // sin^2(theta) / sin^2(theta_max) relative to the cone it was drawn for.
      // g = beta n - 1 is taken as its segment value at lam_min plus the change of
      // the dispersion sum, R(lambda) - R(lam_min) = (s^2 - s_min^2) (k1 / ((k0 - s^2)
      // (k0 - s_min^2)) + k3 / ((k2 - s^2) (k2 - s_min^2))), which FP32 resolves to
      // about 1e-12 in g where R itself would carry 1e-10.
      const float sg = 1000.0f * rcp_fast(lam), sg2 = sg * sg;
      const float dR = (sg2 - p.disp_s2m) *
                       fmaf(p.disp_k1c, rcp_fast(238.0185f - sg2), p.disp_k3c * rcp_fast(57.362f - sg2));
      const float gm = g.q1.w;
      const float gb = fmaxf(fmaf(g.q0.w, dR, gm), 0.f);
      const float c = rcp_fast(1.0f + gb), gg = gb * (gb + 2.0f);
      const float pe = (gg * (c * c)) * (((1.0f + gm) * (1.0f + gm)) * rcp_fast(gm * (gm + 2.0f)));
      emitted = u3 * kU24 < pe;
      inv_pe = rcp_fast(pe);
      cos_t = c;
      sin_t = sqrt_fast(gg) * c;
    }
    // photon on the cone around (0,0,-1), turned onto the track: u = 2 a (a.p) - p
    const float ax = g.q2.x, ay = g.q2.y, az = g.q2.z;
    const float plx = cphi * sin_t, ply = sphi * sin_t, plz = -cos_t;
    const float d2 = 2.0f * fmaf(ax, plx, fmaf(ay, ply, az * plz));
    ux = fmaf(d2, ax, -plx);
    uy = fmaf(d2, ay, -ply);
    uz = fmaf(d2, az, -plz);
  } else {
    // fluorescence (Sec. 4.2.2): isotropic in the lower hemisphere, cos(polar) uniform
    const uint32_t n0 = __float_as_uint(g.q3.w), n1 = g.fl01;
    const uint32_t band = (kk < n0) ? 0u : ((kk < n1) ? 1u : 2u);
    const uint32_t kb = kk - (band == 0u ? 0u : (band == 1u ? n0 : n1));
    const uint4 w = philox_record(g.q3, kb, TAG_FLUOR + band, H.key0, H.key1);
    f = (float)(w.x >> 8);
    const float cz = 1.0f - u24(w.y);
    float sphi, cphi;
    sincospif(2.0f * u24(w.z), &sphi, &cphi);
    const float sz = sqrtf((1.0f - cz) * (1.0f + cz));
    ux = sz * cphi;
    uy = sz * sphi;
    uz = -cz;
    lam = (&s_k->fl.x)[band];
    u3 = (float)(w.w >> 8);
  }
  o.lam = lam;
  o.u3 = u3;
  // detected iff u < p_emit exp(-tau) efficiency / q: compare u / p_emit from here on
  if constexpr (EXT) u3 = u3 * inv_pe;
  o.bin = -1;
  o.tbin = -1;
  o.culled = 0;
  o.t = 0.f;
  o.tau = 0.f;
  o.ux = ux;
  o.uy = uy;
  o.uz = uz;
  const float Px = fmaf(f, g.q1.x, g.q0.x), Py = fmaf(f, g.q1.y, g.q0.y), Pz = fmaf(f, g.q1.z, g.q0.z);
  o.x = Px;
  o.y = Py;
  o.z = Pz;
  if constexpr (EXT && !kMlpTransport<TRANSPORT>) {
    if (!emitted) {  // below the threshold at its wavelength: never emitted
      o.state = kStateNotEmitted;
      return;
    }
  }
  int kb = 0;
  if (TRANSPORT != CPHOT_TRANSPORT_STRAIGHT || p.eff) {
    kb = (int)((lam - H.lam_min) * H.lam_scale);
    kb = min(max(kb, 0), H.n_lam - 1);
  }
  if constexpr (TRANSPORT == CPHOT_TRANSPORT_CURVED || TRANSPORT == kTransportCurvedWalk ||
                TRANSPORT == kTransportCurvedExact || TRANSPORT == kTransportCurvedSurrogate ||
                TRANSPORT == kTransportCurvedTable) {
    // height above the sphere R without subtracting R: (x^2 + y^2 + z (2R + z)) / (|P - C| + R)
    const float Rf = H.Rf;
    const float qz = Pz + Rf;
    const float rq = sqrt_fast(fmaf(Px, Px, fmaf(Py, Py, qz * qz)));
    const float h0 = fmaf(Px, Px, fmaf(Py, Py, Pz * (H.two_Rf + Pz))) * rcp_fast(rq + Rf);
    bool cull = false;  // filter level 3: cannot land on the grid
    if constexpr (TRANSPORT != kTransportCurvedExact) {
      if ((H.cuts & CPHOT_CUT_PHOTON) && uz < 0.f && h0 >= H.h_obs)
        cull = !curved_may_land(p, Px, Py, Pz, ux, uy, uz, rq, h0, core_x, core_y);
    }
    float ym[kMlpOut] = {0.f, 0.f, 0.f, 0.f};
    bool use_mlp = false;
    float c0 = 0.f;    // cos of the local zenith angle (angle between -u and the upward radial)
    float leg = 0.f;   // straight path inside the start shell, down to its lower boundary
    int j0 = 0;        // start shell
    if constexpr (TRANSPORT == kTransportCurvedSurrogate) {
      const float irq = rcp_fast(rq);
      c0 = -fmaf(ux, Px * irq, fmaf(uy, Py * irq, uz * (qz * irq)));
      const bool alive = valid && emitted && (uz < 0.f) && (h0 >= H.h_obs) && !cull;
      // the network starts at the start shell's lower boundary R + h_b (the photon is
      // straight inside its homogeneous start shell); a start inside the observation
      // shell is straight all the way (h_b = h_obs, nothing left to correct)
      j0 = min((int)(h0 * H.inv_dh), H.n_layers - 1);
      const bool in_obs = j0 <= H.obs_layer;
      const float h_b = in_obs ? H.h_obs : (float)j0 * H.dh;
      const float rc0 = (Rf + h0) * c0;
      const float dJ = (h0 - h_b) * (2.0f * Rf + h0 + h_b);  // r0^2 - r_b^2
      const float gb = fmaf(rc0, rc0, -dJ);                   // r_b^2 cos^2 at the boundary
      const bool reach = c0 > 0.f && gb > 0.f;
      const float sgb = sqrt_fast(fmaxf(gb, 0.f));
      leg = reach ? dJ * rcp_fast(rc0 + sgb) : 0.f;
      float xin[kMlpIn] = {h_b, sgb * rcp_fast(Rf + h_b), atan2f(uy, ux),
                           H.lam_min + ((float)kb + 0.5f) * p.lam_step, H.h_obs};
      use_mlp = alive && reach && (in_obs || mlp_in_domain(s_img, xin));
      if (!use_mlp || in_obs) {
#pragma unroll
        for (int q = 0; q < kMlpIn; ++q) xin[q] = s_img->in_lo[q];  // finite filler for lanes that do not use it
      }
      // the whole wave evaluates the network together, or skips it when no lane needs it
      if (__ballot(use_mlp && !in_obs)) mlp_forward_wave(s_img, xin, ym, s_stage);
      if (in_obs) {
#pragma unroll
        for (int q = 0; q < kMlpOut; ++q) ym[q] = 0.f;
      }
      if (EXT && !emitted) {
        o.state = kStateNotEmitted;
        return;
      }
    }
    if (!(uz < 0.f)) {
      o.state = kStateUp;
      return;
    }
    if (h0 < H.h_obs) {
      o.state = kStateOutside;
      return;
    }
    if (cull) {
      o.state = kStateOutside;
      o.culled = 1;
      return;
    }
    if constexpr (TRANSPORT == kTransportCurvedTable) {
      // correction interpolated from the table (Sec. 4.4.1), in the start shell
      const float irq = rcp_fast(rq);
      c0 = -fmaf(ux, Px * irq, fmaf(uy, Py * irq, uz * (qz * irq)));
      float4 v;
      const float tz = sqrt_fast(fmaxf((1.0f - c0) * (1.0f + c0), 0.f)) * rcp_fast(c0);
      use_mlp = c0 > 0.f && table_lookup(p.ctab, min((int)(h0 * H.inv_dh), H.n_layers - 1), h0, tz, v);
      const float2 sp = s_lam[kb];
      ym[0] = v.x;
      ym[2] = v.y;
      ym[3] = -fmaf(v.z, sp.x, v.w * sp.y);
    }
    CurvedWalk cw;
    if (use_mlp) {
      // straight chord to the sphere R + h_obs (cancellation-free root), its
      // central angle, plus the predicted extra ground distance, offset across,
      // optical path excess and log T (the network predicts them per metre of chord)
      const float r0 = Rf + h0, r1 = H.r_obs;
      const float s0 = sqrt_fast(fmaxf((1.0f - c0) * (1.0f + c0), 0.f));
      const float drs = (h0 - H.h_obs) * (r0 + r1);
      const float rc = r0 * c0;
      const float s_ch = drs * rcp_fast(rc + sqrt_fast(fmaf(rc, rc, -drs)));
      const float xs = s_ch * s0 * rcp_fast(r1);
      const float psi_s = fmaf(xs * xs * (1.0f / 6.0f), xs, xs);
      // the network's outputs are per metre of the chord from the start shell's lower
      // boundary (the same straight line, shortened by the leg inside the start
      // shell, whose optical depth and n - 1 are added exactly); the table's are absolute
      const float scale = (TRANSPORT == kTransportCurvedTable) ? 1.0f : s_ch - leg;
      const float psi = fmaf(ym[0] * scale, rcp_fast(r1), psi_s);
      curved_arrival(Rf, H.h_obs, r1, Px, Py, Pz, h0, ux, uy, uz, psi, ym[1] * scale, cw.ax, cw.ay, cw.az);
      const float4 Lj = s_lay[j0];
      cw.tau = fmaf(fmaf(Lj.z, s_lam[kb].x, Lj.w * s_lam[kb].y), leg, -ym[3] * scale);
      cw.arrived = 1;
      cw.geo = 0.f;
      cw.opt = 0.f;
      if constexpr (NEED_TIME) {
        // delay = chord (1 - u.a) + excess - (arrival - chord end) . a
        const float gx = ux - axx, gy = uy - axy, gz = uz - axz;
        const double ex = (double)Px + (double)s_ch * ux, ey = (double)Py + (double)s_ch * uy,
                     ez = (double)Pz + (double)s_ch * uz;
        const float shift = (float)((cw.ax - ex) * axx + (cw.ay - ey) * axy + (cw.az - ez) * axz);
        cw.geo = fmaf(s_ch * 0.5f, fmaf(gx, gx, fmaf(gy, gy, gz * gz)), -shift);
        cw.opt = fmaf(Lj.x, leg, ym[2] * scale);
      }
    } else {
      if constexpr (TRANSPORT == kTransportCurvedSurrogate || TRANSPORT == kTransportCurvedTable) {
        o.state = kStateDeferred;  // outside the domain: traced exactly in a compacted pass
        return;
      }
      if constexpr (TRANSPORT == CPHOT_TRANSPORT_CURVED || TRANSPORT == kTransportCurvedExact) {
        // closed-form shell sums; rays outside their domain are walked in a compacted pass
        if (!curved_series<NEED_TIME>(s_lay, H, p, s_k->rc, s_lam[kb], Px, Py, Pz, rq, h0, ux, uy, uz, axx, axy, axz, cw)) {
          o.state = kStateDeferred;
          return;
        }
      } else {
        curved_walk<NEED_TIME>(s_lay, s_lam[kb], p, Px, Py, Pz, h0, ux, uy, uz, axx, axy, axz, cw);
      }
    }
    o.x = (float)cw.ax;
    o.y = (float)cw.ay;
    o.z = (float)cw.az;
    o.tau = cw.tau;
    if constexpr (NEED_TIME) o.t = (cw.geo + cw.opt) * (1.0f / kCmPerNs);
    if (!cw.arrived) {
      o.state = kStateOutside;
      return;
    }
    if (!(u3 < survival_threshold(s_eff, cw.tau, kb, g.inv_q))) {
      o.state = kStateAbsorbed;
      return;
    }
    // bins in the tangent plane at the core, in FP64
    const double fxc = floor((cw.ax - S.x64) * H.inv_cell64), fyc = floor((cw.ay - S.y64) * H.inv_cell64);
    if (!(fxc >= 0.0 && fyc >= 0.0 && fxc < H.nx64 && fyc < H.ny64)) {
      o.state = kStateOutside;
      return;
    }
    o.state = 0;
    o.ix = (int)fxc;
    o.iy = (int)fyc;
    o.bin = o.iy * H.nx + o.ix;
    return;
  } else {
  float ym[kMlpOut] = {0.f, 0.f, 0.f, 0.f};
  bool use_mlp = false;
  float h_b = Pz;   // the network's start: the lower boundary of the start layer (no leg otherwise)
  int j0 = 0;       // start layer
  if constexpr (TRANSPORT == CPHOT_TRANSPORT_SURROGATE) {
    const bool alive = valid && emitted && (uz < 0.f) && (Pz >= H.h_obs);
    // straight inside the homogeneous start layer; the network takes over at its lower
    // boundary; a start inside the observation layer is straight all the way
    j0 = min((int)(Pz * H.inv_dh), H.n_layers - 1);
    const bool in_obs = j0 <= H.obs_layer;
    h_b = in_obs ? H.h_obs : (float)j0 * H.dh;
    float xin[kMlpIn] = {h_b, -uz, atan2f(uy, ux),
                         H.lam_min + ((float)kb + 0.5f) * p.lam_step, H.h_obs};
    use_mlp = alive && (in_obs || mlp_in_domain(s_img, xin));
    if (!use_mlp || in_obs) {
#pragma unroll
      for (int q = 0; q < kMlpIn; ++q) xin[q] = s_img->in_lo[q];  // finite filler for lanes that do not use it
    }
    // the whole wave evaluates the network together, or skips it when no lane needs it
    if (__ballot(use_mlp && !in_obs)) mlp_forward_wave(s_img, xin, ym, s_stage);
    if (in_obs) {
#pragma unroll
      for (int q = 0; q < kMlpOut; ++q) ym[q] = 0.f;
    }
    if (EXT && !emitted) {
      o.state = kStateNotEmitted;
      return;
    }
  }
  if (!(uz < 0.f)) {
    o.state = kStateUp;
    return;
  }
  if (Pz < H.h_obs) {
    o.state = kStateOutside;
    return;
  }
  if constexpr (DETECTOR == CPHOT_DETECTOR_SPHERES && !kMlpTransport<TRANSPORT>) {
    if ((H.cuts & CPHOT_CUT_PHOTON) && !photon_may_hit(p, Px, Py, Pz, ux, uy, uz, core_x, core_y)) {
      o.state = kStateOutside;  // filter level 3: cannot reach a sphere
      o.culled = 1;
      return;
    }
  }
  if constexpr (DETECTOR == CPHOT_DETECTOR_GRID && !kMlpTransport<TRANSPORT>) {
    if ((H.cuts & CPHOT_CUT_PHOTON) && !grid_may_hit(p, Px, Py, Pz, ux, uy, uz, core_x, core_y)) {
      o.state = kStateOutside;  // filter level 3: cannot land on the grid
      o.culled = 1;
      return;
    }
  }
  if constexpr (TRANSPORT == CPHOT_TRANSPORT_TABLE) {
    // correction interpolated from the table (Sec. 4.4.1), in the start layer
    float4 v;
    const float tz = sqrtf(fmaf(ux, ux, uy * uy)) / -uz;
    use_mlp = table_lookup(p.ctab, min((int)(Pz * H.inv_dh), H.n_layers - 1), Pz, tz, v);
    const float2 sp = s_lam[kb];
    ym[0] = v.x;
    ym[2] = v.y;
    ym[3] = -fmaf(v.z, sp.x, v.w * sp.y);
  }
  float x, y, z;     // start of the final leg
  float vx, vy, vz;  // direction of the final leg
  float tau = 0.f, geo = 0.f, opt = 0.f;
  float last_delta = 0.f, last_ext = 0.f;
  bool series = false;  // the path sums came from the closed forms, without those of the time
  if constexpr (TRANSPORT != CPHOT_TRANSPORT_STRAIGHT) {
    if (TRANSPORT == CPHOT_TRANSPORT_LAYERED || !use_mlp) {
      if constexpr (TRANSPORT == CPHOT_TRANSPORT_SURROGATE || TRANSPORT == CPHOT_TRANSPORT_TABLE) {
        o.state = kStateDeferred;  // outside the domain: traced exactly in a compacted pass
        return;
      }
      LayerWalk lw;
      const int j0 = min((int)(Pz * H.inv_dh), H.n_layers - 1);
      // closed-form sums where the series holds, the crossing loop elsewhere
      series = j0 > H.obs_layer && fmaf(ux, ux, uy * uy) <= H.series_tmax * (uz * uz);
      if (series)
        layer_series<NEED_TIME && ROWS>(s_lay, H.moments, s_lam[kb], H.dh, j0, H.obs_layer, Px, Py, Pz, ux, uy, uz,
                                        axx, axy, axz, lw);
      else
        layer_walk<NEED_TIME>(s_lay, s_lam[kb], H.dh, j0, H.obs_layer, Px, Py, Pz, ux, uy, uz, axx, axy,
                                     axz, lw);
      x = lw.x;
      y = lw.y;
      z = lw.z;
      vx = lw.vx;
      vy = lw.vy;
      vz = lw.vz;
      tau = lw.tau;
      geo = lw.geo;
      opt = lw.opt;
      last_delta = lw.last_delta;
      last_ext = lw.last_ext;
    } else {
      // straight line to the observation level plus the predicted correction:
      // landing (dx, dy), optical path excess e and log T; the delay after the
      // plane front is [l (1 - u.a) + e - (dx a_x + dy a_y)] / c
      const float s_pl = (H.h_obs - Pz) / uz;
      // the predicted offset is along / across the photon's horizontal direction
      const float sh = sqrtf(fmaf(ux, ux, uy * uy));
      const float hx = sh > 0.f ? ux / sh : 1.f, hy = sh > 0.f ? uy / sh : 0.f;
      const float odx = fmaf(ym[0], hx, -ym[1] * hy), ody = fmaf(ym[0], hy, ym[1] * hx);
      x = fmaf(s_pl, ux, Px) + odx;
      y = fmaf(s_pl, uy, Py) + ody;
      z = H.h_obs;
      vx = ux;
      vy = uy;
      vz = uz;
      // the leg inside the start layer down to the network's start h_b, exactly, and
      // for the table its absolute sums; the network predicts what refraction adds to
      // the straight line's own sums below h_b (full layers from the layer-sum
      // moments, the observation layer's span directly)
      const float ic = 1.0f / -uz;
      const float leg = (Pz - h_b) * ic;
      const float4 Lj = s_lay[j0];
      const float2 sp = s_lam[kb];
      float tau_s = 0.f, opt_s = 0.f;
      if constexpr (TRANSPORT == CPHOT_TRANSPORT_SURROGATE) {
        if (j0 > H.obs_layer) {
          const float4* mr = H.moments + 5 * j0;
          const float4 Lo = s_lay[H.obs_layer];
          const float top = (float)(H.obs_layer + 1) * H.dh - H.h_obs;
          tau_s = ic * fmaf(sp.x, mr[2].w, fmaf(sp.y, mr[3].z, fmaf(Lo.z, sp.x, Lo.w * sp.y) * top));
          opt_s = ic * fmaf(Lo.x, top, mr[2].x);
        }
      }
      tau = fmaf(fmaf(Lj.z, sp.x, Lj.w * sp.y), leg, tau_s - ym[3]);
      if constexpr (NEED_TIME) {
        const float gx = ux - axx, gy = uy - axy, gz = uz - axz;
        geo = s_pl * 0.5f * (gx * gx + gy * gy + gz * gz) - (odx * axx + ody * axy);
        opt = fmaf(Lj.x, leg, opt_s + ym[2]);
      }
      const float4 L = s_lay[H.obs_layer];
      last_delta = L.x;
      last_ext = fmaf(L.z, sp.x, L.w * sp.y);
    }
  } else {
    x = Px;
    y = Py;
    z = Pz;
    vx = ux;
    vy = uy;
    vz = uz;
  }
  // final straight leg: crossing of the observation level
  const float s_plane = (H.h_obs - z) * rcp_fast(vz);
  const float Qx = fmaf(s_plane, vx, x), Qy = fmaf(s_plane, vy, y);
  float s_end = s_plane;
  int32_t bin = -1;
  if constexpr (DETECTOR == CPHOT_DETECTOR_GRID) {
    const float fxc = floorf((Qx - S.x0) * H.inv_cell), fyc = floorf((Qy - S.y0) * H.inv_cell);
    if (fxc >= 0.f && fyc >= 0.f && fxc < (float)H.nx && fyc < (float)H.ny) {
      o.ix = (int)fxc;
      o.iy = (int)fyc;
      bin = o.iy * H.nx + o.ix;
    }
  } else {
    const float cx0 = S.x0, cy0 = S.y0;
    const float fi = floorf((Qx - cx0) * H.inv_pitch + 0.5f), fj = floorf((Qy - cy0) * H.inv_pitch + 0.5f);
    if (fi >= 0.f && fj >= 0.f && fi < (float)H.snx && fj < (float)H.sny) {
      const float qx = Qx - (cx0 + fi * H.pitch), qy = Qy - (cy0 + fj * H.pitch);
      const float b = qx * vx + qy * vy;  // q_z = 0 on the observation level
      const float cc = qx * qx + qy * qy - H.radius * H.radius;
      const float disc = b * b - cc;
      if (disc >= 0.f) {
        s_end = s_plane + (-b - sqrt_fast(disc));
        bin = (int)fj * H.snx + (int)fi;
      }
    }
  }
  const float ex = fmaf(s_end, vx, x), ey = fmaf(s_end, vy, y), ez = fmaf(s_end, vz, z);
  float inv_uz = 0.f, Xe = 0.f, X_end = 0.f;
  if constexpr (TRANSPORT != CPHOT_TRANSPORT_STRAIGHT) {
    tau = fmaf(last_ext, s_end, tau);
  } else {
    // straight line in a planar atmosphere: closed forms over the height span
    inv_uz = -1.0f / vz;  // 1/|u_z|
    Xe = fmaf(f, g.dX, g.q2.w);
    X_end = p.X_obs;
    if constexpr (DETECTOR == CPHOT_DETECTOR_SPHERES) {
      if (p.profile == CPHOT_PROFILE_LINSLEY5) X_end = depth_f(*s_k, ez);
    }
    if (p.has_ray) {
      const float r = 400.0f / lam;
      const float r2 = r * r;
      tau = (X_end - Xe) * inv_uz * (r2 * r2 * p.inv_ray400);
    }
    if (p.has_aer) {
      const float taua = p.aer_tau350 * __powf(lam * (1.0f / 350.0f), -p.aer_ang);
      tau = fmaf(taua * (__expf(-ez * p.aer_inv_h) - __expf(-Pz * p.aer_inv_h)), inv_uz, tau);
    }
  }
  // Delay after the plane front. Few records are binned (of the telescope array's 1 in
  // 170), so its sums are formed where they are used, in a third of the waves (1e6
  // segments 130 -> 127 us).
  auto delay = [&]() {
    const float gx = vx - axx, gy = vy - axy, gz = vz - axz;
    const float g2 = gx * gx + gy * gy + gz * gz;
    if constexpr (TRANSPORT == CPHOT_TRANSPORT_STRAIGHT) {
      geo = s_end * 0.5f * g2;
      opt = opt_integral(p, ez, Pz, X_end, Xe) * inv_uz;
    } else {
      if (!ROWS && series) {
        LayerWalk lw;
        layer_series<true>(s_lay, H.moments, s_lam[kb], H.dh, min((int)(Pz * H.inv_dh), H.n_layers - 1), H.obs_layer, Px,
                           Py, Pz, ux, uy, uz, axx, axy, axz, lw);
        geo = lw.geo;
        opt = lw.opt;
      }
      geo = fmaf(s_end, 0.5f * g2, geo);
      opt = fmaf(last_delta, s_end, opt);
    }
    return (geo + opt) * (1.0f / kCmPerNs);
  };
  o.x = ex;
  o.y = ey;
  o.z = ez;
  o.tau = tau;
  if constexpr (NEED_TIME && ROWS) o.t = delay();
  if (!(u3 < survival_threshold(s_eff, tau, kb, g.inv_q))) {
    o.state = kStateAbsorbed;
    return;
  }
  if (bin < 0) {
    o.state = kStateOutside;
    return;
  }
  o.state = 0;
  o.bin = bin;
  if constexpr (DETECTOR == CPHOT_DETECTOR_SPHERES) {
    if (H.n_t > 0) {
      const float tb = floorf((ROWS ? o.t : delay()) * H.inv_dt);
      o.tbin = tb < 0.f ? 0 : (tb >= (float)H.n_t ? H.n_t : (int)tb);
    }
  }
  }
}

}  // namespace

// Shower of segment i: the largest s with offsets[s] <= i.
__device__ __forceinline__ int shower_of(const KParams& p, int64_t i) {
  if (p.n_showers <= 1) return 0;
  int lo = 0, hi = p.n_showers;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (p.offsets[mid] <= i) lo = mid; else hi = mid;
  }
  return lo;
}

// The kernel's arguments, read anew: the address passes through a statement that the
// compiler cannot see through, so that values used once per record are loaded (scalar
// cache) where they are used. Hoisted out of the record loop they overflow the scalar
// registers by over a hundred, and each use reads them back with a lane read.
__device__ __forceinline__ const KParams& fresh_params() {
  auto q = __builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(q));
  return *(const KParams*)q;
}

// A value that is the same in every lane, in a scalar register.
__device__ __forceinline__ float uniform(float v) {
  return __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(v)));
}

__device__ __forceinline__ double uniform(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32));
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Adds w photons to element b of the global bins.
__device__ __forceinline__ void add_bin(const KParams& p, int64_t b, uint32_t w) {
  if (p.bins_f64) atomicAdd(reinterpret_cast<double*>(p.bins) + b, (double)(float)w);
  else if (p.bins_u64) atomicAdd(reinterpret_cast<unsigned long long*>(p.bins) + b, (unsigned long long)w);
  else atomicAdd(reinterpret_cast<uint32_t*>(p.bins) + b, w);
}

// A block's LDS window: the rectangle of grid cells (or the sphere array) it holds.
struct Window {
  int w, h, x0, y0;
};

// The window of a shower's grid. The launch gives the rectangle, or only its area
// (hist_auto): then the sides are in the ratio of the extents of a round spot, cast along
// the shower axis, on the ground (1 + (axis_x / axis_z)^2 and the same in y, squared), and
// the rectangle's centre is the grid's plus the caller's shift, inside the grid. Photons of a
// shower inclined by 60 degrees that miss a square of the same area cost a device atomic each.
__device__ __forceinline__ Window shower_window(const KParams& p, int sh) {
  Window w = {p.hist_w, p.hist_h, p.hist_x0, p.hist_y0};
  if (p.hist_auto) {
    const double* g = p.geom + 5 * (int64_t)sh;
    const float ex = (float)(g[2] / g[4]), ey = (float)(g[3] / g[4]);
    const float area = (float)p.hist_auto;
    const float side = sqrtf(area * sqrtf(fmaf(ex, ex, 1.0f) / fmaf(ey, ey, 1.0f)));
    // an axis along the ground (or no number) gives the whole width
    w.w = side < (float)p.nx ? max((int)side, 1) : p.nx;
    w.h = min(p.hist_auto / w.w, p.ny);
    if (w.h == p.ny) w.w = min(p.hist_auto / w.h, p.nx);
    w.w = __builtin_amdgcn_readfirstlane(w.w);
    w.h = __builtin_amdgcn_readfirstlane(w.h);
    w.x0 = min(max((p.nx - w.w) / 2 + p.hist_x0, 0), p.nx - w.w);
    w.y0 = min(max((p.ny - w.h) / 2 + p.hist_y0, 0), p.ny - w.h);
  }
  return w;
}

// Adds the LDS window of shower `sh` (record counts) to the global bins with
// the bunch weight, and clears it. Called by the whole block. Of a grid's window a wave
// takes whole rows, so that its atomics fall on consecutive cells; the sphere array and its
// leading time bins lie in LDS as they are numbered, so the block walks them lane by lane (a
// sphere per wave and turn took 105 us for 10,000 spheres in a block of 256, whatever was
// counted, 14 us lane by lane).
template <int BS, int DETECTOR>
__device__ void flush_window(const KParams& p, uint32_t* s_hist, const Window& win, int sh) {
  auto add = [&](int64_t gb, uint32_t v) {
    const unsigned long long w = (unsigned long long)v * (unsigned long long)p.bunch;
    if (p.bins_f64) atomicAdd(reinterpret_cast<double*>(p.bins) + gb, (double)w);
    else if (p.bins_u64) atomicAdd(reinterpret_cast<unsigned long long*>(p.bins) + gb, w);
    else atomicAdd(reinterpret_cast<uint32_t*>(p.bins) + gb, (uint32_t)w);
  };
  if constexpr (DETECTOR == CPHOT_DETECTOR_GRID) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, row = p.nx;
    const int64_t base = (int64_t)sh * row * p.ny;
    for (int ly = wave; ly < win.h; ly += BS / 64) {
      for (int lx = lane; lx < win.w; lx += 64) {
        const uint32_t v = s_hist[ly * win.w + lx];
        if (v) {
          add(base + (int64_t)(win.y0 + ly) * row + (win.x0 + lx), v);
          s_hist[ly * win.w + lx] = 0u;
        }
      }
    }
  } else {
    const int n = win.w * win.h, nt = n * p.hist_tw;
    const int64_t base = (int64_t)sh * n;
    for (int b = threadIdx.x; b < n; b += BS) {
      const uint32_t v = s_hist[b];
      if (v) {
        add(base + b, v);
        s_hist[b] = 0u;
      }
    }
    for (int b = threadIdx.x; b < nt; b += BS) {
      const uint32_t v = s_hist[n + b];
      if (v) {
        const int sph = b / p.hist_tw, tb = b - sph * p.hist_tw;
        atomicAdd(p.thist + (base + sph) * (p.n_t + 1) + tb, v * (uint32_t)p.bunch);
        s_hist[n + b] = 0u;
      }
    }
  }
}

// Waves per SIMD the register allocation must leave room for: four (128 registers) for
// the exact tracers, whose time falls with the waves up to there (inclined step with a
// window that catches its photons: 26.6, 17.7 and 14.4 ms at two, three and four); the
// network's activations allow two, three in the block of 768 with a few values of the
// tile set-up in scratch.
template <int BS, int T>
constexpr int kMinWaves = !kMlpTransport<T> ? 4 : BS == 768 ? 3 : 2;

// EXT: Poisson record counts and the dispersive spectrum (its per-record angle and
// emission decision), compiled only into the kernels that run them: as runtime
// branches their registers cost the default path spills and about a tenth of its
// time.
template <int BS, int TRANSPORT, int DETECTOR, int MODE, bool EXT>
__global__ __launch_bounds__(BS, (kMinWaves<BS, TRANSPORT>)) void k_propagate(KParams p) {
  constexpr bool kTime = (DETECTOR == CPHOT_DETECTOR_SPHERES) || (MODE == MODE_RECORDS);
  constexpr bool kLayers = (TRANSPORT != CPHOT_TRANSPORT_STRAIGHT);
  constexpr bool kMlp = (TRANSPORT == CPHOT_TRANSPORT_SURROGATE || TRANSPORT == kTransportCurvedSurrogate);
  // transports that defer some records to the exact tracer (compaction queue)
  constexpr bool kDefer = kMlp || TRANSPORT == CPHOT_TRANSPORT_TABLE || TRANSPORT == kTransportCurvedTable ||
                          TRANSPORT == CPHOT_TRANSPORT_CURVED;
  constexpr bool kRecords = MODE == MODE_RECORDS;
  constexpr int kWaves = BS / 64;
  // exact transport behind a surrogate: records outside the network's domain
  constexpr int kExact =
      (TRANSPORT == CPHOT_TRANSPORT_SURROGATE || TRANSPORT == CPHOT_TRANSPORT_TABLE)       ? CPHOT_TRANSPORT_LAYERED
      : (TRANSPORT == kTransportCurvedSurrogate || TRANSPORT == kTransportCurvedTable) ? kTransportCurvedExact
      : (TRANSPORT == CPHOT_TRANSPORT_CURVED)                                               ? kTransportCurvedWalk
                                                                                            : TRANSPORT;
  // the closed-form sums behind a curved network or table defer once more, to the shell walk
  constexpr int kQueues = kExact == kTransportCurvedExact ? 2 : 1;
  // per-segment state for the record loop (SegState), 64 slots per wave
  __shared__ float4 s_q0[BS], s_q1[BS], s_q2[BS], s_q3[BS];
  __shared__ uint32_t s_fl01[BS];
  __shared__ float2 s_dx[kLayers ? 1 : BS];
  // record dumps: the segment's global id, its first record's place, its Cherenkov records
  __shared__ ulonglong2 s_rec[kRecords ? BS : 1];
  __shared__ uint32_t s_nch[kRecords ? BS : 1];
  constexpr int kRowsAtOnce = 32;
  __shared__ uint4 s_row[kRecords ? kWaves * 4 * kRowsAtOnce : 1];
  __shared__ float4 s_lay[kLayers ? kMaxLayers : 1];
  __shared__ float2 s_lam[kLayers ? kMaxLambdaBins : 1];
  __shared__ uint4 s_imgw[kMlp ? sizeof(MlpImage) / 16 : 1];
  // compaction queue of deferred records (slot + 64 kind + 128 index), 64 entries per
  // wave: the wave traces what it holds when a round's records would not fit
  __shared__ uint32_t s_queue[kDefer ? kQueues * BS : 1];
  __shared__ uint4 s_mlpx[kMlp ? BS : 1];  // per-wave staging of the network's inputs and outputs
  __shared__ KConst s_k;
  __shared__ float s_eff[kMaxLambdaBins];  // detector efficiency per wavelength bin, times 2^24
  __shared__ unsigned long long s_cnt[CPHOT_NCOUNTERS];
  // Optional LDS window of the grid, or the whole sphere array (record counts of
  // one shower at a time). With it each block walks a contiguous range of tiles,
  // so the window changes shower only a few times per block; records outside the
  // window, or of another shower than the window's, go to the global bins
  // directly. Without it every hit is a device atomic, and hits on one sphere
  // serialise on its cache line.
  extern __shared__ uint32_t s_hist[];
  __shared__ unsigned long long s_since;  // records counted in the window since it was clear, at most
  __shared__ uint32_t s_next;             // next unit of the block's run, from its first
  // segments of the run's shower (kept where batches run; in the curved kernels the few
  // registers it takes cost 1 %)
  constexpr bool kRange = DETECTOR == CPHOT_DETECTOR_GRID && (TRANSPORT == CPHOT_TRANSPORT_STRAIGHT || TRANSPORT == CPHOT_TRANSPORT_LAYERED);
  __shared__ int64_t s_range[kRange ? 2 : 1];
  const int n_hist = MODE == MODE_PROPAGATE ? p.hist_words : 0;
  const int tid = threadIdx.x, lane = tid & 63, wbase = tid & ~63;

  if constexpr (kLayers) {
    for (int i = tid; i < p.n_layers; i += BS) s_lay[i] = p.layers[i];
    for (int i = tid; i < p.n_lam; i += BS) s_lam[i] = p.lambins[i];
  }
  if constexpr (kMlp) {
    const uint4* src = reinterpret_cast<const uint4*>(p.mlp);
    for (int i = tid; i < (int)(sizeof(MlpImage) / 16); i += BS) s_imgw[i] = src[i];
  }
  load_kconst(p, s_k, tid);
  for (int i = tid; i < kMaxLambdaBins; i += BS)
    s_eff[i] = ((p.eff && i < p.n_lam) ? (float)p.eff[i] : 1.0f) * 16777216.0f;
  for (int i = tid; i < n_hist; i += BS) s_hist[i] = 0u;
  if (tid < CPHOT_NCOUNTERS) s_cnt[tid] = 0ull;
  if (tid == 0) s_since = 0ull;
  __syncthreads();
  const Tables T = {s_lay, s_lam, reinterpret_cast<const MlpImage*>(s_imgw), &s_k, s_eff,
                    s_mlpx + (kMlp ? wbase : 0)};

  constexpr int kKept = (TRANSPORT == CPHOT_TRANSPORT_STRAIGHT || TRANSPORT == CPHOT_TRANSPORT_LAYERED ||
                         TRANSPORT == CPHOT_TRANSPORT_TABLE)
                            ? 2
                            : kMlp ? 1 : 0;
  const Hot<kKept> H(p);

  // Units of work: a tile of 64 segments, or with sub_shift one of the 2^sub_shift equal
  // shares of its record rounds. With an LDS histogram the block walks a contiguous range
  // of them, one run per shower; its waves draw units from the run as they finish, the
  // last ones of a run in halves, and the ranges fall linearly with the block index where
  // more blocks are launched than run at a time. Without, the waves of the grid take units
  // in turn.
  const int64_t n_units = ((p.n + 63) >> 6) << p.sub_shift;
  int64_t u_first = 0, u_end = n_units;
  if (n_hist) {
    const KParams& p = fresh_params();
    auto edge = [&](uint32_t b) {
      const double x = (double)b / (double)gridDim.x;
      return (int64_t)((double)n_units * (x + (double)p.taper * x * (1.0 - x)));
    };
    u_first = edge(blockIdx.x);
    u_end = blockIdx.x + 1 == gridDim.x ? n_units : edge(blockIdx.x + 1);
  }
  int win_sh = -1;
  Window win = {0, 0, 0, 0};
  for (int64_t run = u_first, run_end; run < u_end; run = run_end) {
    run_end = u_end;
    if (n_hist) {
      const KParams& p = fresh_params();
      const int sh = shower_of(p, (run >> p.sub_shift) << 6);
      if (sh + 1 < p.n_showers) run_end = min(u_end, ((p.offsets[sh + 1] + 63) >> 6) << p.sub_shift);
      if (run != u_first) {
        __syncthreads();
        flush_window<BS, DETECTOR>(p, s_hist, win, win_sh);
        __syncthreads();
      }
      win_sh = sh;
      win = shower_window(p, sh);
      if (tid == 0) {
        s_next = 0u;
        s_since = 0ull;
        if constexpr (kRange) {
          s_range[0] = p.n_showers > 1 ? p.offsets[sh] : 0;
          s_range[1] = sh + 1 < p.n_showers ? p.offsets[sh + 1] : p.n;
        }
      }
      __syncthreads();
    }
    for (int64_t turn = (int64_t)blockIdx.x * kWaves + (tid >> 6);; turn += (int64_t)gridDim.x * kWaves) {
      const KParams& p = fresh_params();
      int64_t unit = turn;
      uint32_t half = 2;  // 0, 1: this half of the unit's rounds; 2: all
      if (n_hist) {
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&s_next, 1u);
        at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
        const uint32_t n_run = (uint32_t)(run_end - run), whole = n_run - min((uint32_t)p.tail_units, n_run);
        // A SIMD issues its oldest wave first, and equal blocks of one CU ended a third apart;
        // the more units a block has left (in quarters of a mean block's), the higher its
        // waves' priority (telescope array 127 -> 113 us; all blocks above 512 are alone on
        // their CU).
        if constexpr (BS <= 512) {
          const float left = (float)(uint32_t)max((int64_t)0, u_end - run - at) * p.inv_share4;
          const int rank = __builtin_amdgcn_readfirstlane((int)left);
          if (rank <= 0) __builtin_amdgcn_s_setprio(0);
          else if (rank == 1) __builtin_amdgcn_s_setprio(1);
          else if (rank == 2) __builtin_amdgcn_s_setprio(2);
          else __builtin_amdgcn_s_setprio(3);
        }
        if (at >= whole) {
          half = (at - whole) & 1u;
          at = whole + ((at - whole) >> 1);
        }
        unit = run + at;
      }
      if (unit >= run_end) break;
      const int64_t tile = unit >> p.sub_shift;
      int sub = p.sub_shift;
      uint32_t share = (uint32_t)unit & ((1u << sub) - 1u);
      if (half < 2u) {
        share = 2u * share + half;
        ++sub;
      }
      // ---- 1. the tile's segments, one per lane
      const int64_t i = (tile << 6) + lane;
      uint32_t n_ch = 0, n_fl = 0;
      float4 q0 = make_float4(0.f, 0.f, 0.f, 0.f), q1 = q0, q2 = q0, q3 = q0;
      uint2 fl_n = make_uint2(0u, 0u);
      float inv_q = 1.f;
      uint32_t key = kMaxLayers;  // segments without records sort last
      int status = 0;
      uint32_t cut1 = 0;
      uint32_t sh_of = 0;
      float dXs = 0.f;
      uint64_t id = 0;
      if (i < p.n) {
        const float fx0 = p.x0[i], fy0 = p.y0[i], fz0 = p.z0[i], fx1 = p.x1[i], fy1 = p.y1[i], fz1 = p.z1[i];
        id = p.first_id + (uint64_t)i * p.id_stride;
        SegResult r = segment_setup<EXT>(p, fx0, fy0, fz0, fx1, fy1, fz1, p.beta[i], p.charge[i],
                                         p.dedx ? p.dedx[i] : 0.0f, id);
        if constexpr (MODE == MODE_PROPAGATE && DETECTOR == CPHOT_DETECTOR_SPHERES && !kMlpTransport<TRANSPORT>) {
          if ((p.cuts & CPHOT_CUT_TRACK) && r.n > 0) {
            const double* gc = p.geom + 5 * shower_of(p, i);
            if (!track_may_hit(p, fx0, fy0, fz0, fx1, fy1, fz1, r.cos_t, r.sin_t, (float)gc[0], (float)gc[1])) {
              cut1 = (uint32_t)r.n;  // filter level 1: no photon of the cone can reach a sphere
              r.n = 0;
            }
          }
        }
        status = r.status;
        n_ch = (uint32_t)r.n;
        fl_n = make_uint2((uint32_t)r.nf[0], (uint32_t)(r.nf[0] + r.nf[1]));
        inv_q = r.inv_q;
        n_fl = (uint32_t)(r.nf[0] + r.nf[1] + r.nf[2]);
        if (n_ch + n_fl) {
          // nearly always the run's shower; the search is a chain of dependent loads (3e6
          // segments in 16 showers 1,112 us with it for every segment, 1,094 without)
          if (kRange && n_hist && i >= s_range[0] && i < s_range[1]) sh_of = (uint32_t)win_sh;
          else sh_of = (uint32_t)shower_of(p, i);
          float X0 = 0.f;
          if (!kLayers && p.profile == CPHOT_PROFILE_LINSLEY5) {
            X0 = depth_f(s_k, fz0);
            dXs = (depth_f(s_k, fz1) - X0) * kU24;
          }
          const bool disp = EXT && p.spectrum == CPHOT_SPECTRUM_DISPERSIVE;
          const uint3 ph = philox_segment((uint32_t)id, (uint32_t)(id >> 32), p.key0, p.key1);
          q0 = make_float4(fx0, fy0, fz0, disp ? r.disp_a : r.cos_t);
          q1 = make_float4((fx1 - fx0) * kU24, (fy1 - fy0) * kU24, (fz1 - fz0) * kU24, disp ? r.disp_gm : r.sin_t);
          q2 = make_float4(r.a0, r.a1, r.a2, kLayers ? inv_q : X0);
          q3 = make_float4(__uint_as_float(ph.x), __uint_as_float(ph.y), __uint_as_float(ph.z),
                           __uint_as_float(fl_n.x));
          if constexpr (kLayers) key = (uint32_t)min(max((int)(0.5f * (fz0 + fz1) * p.inv_dh), 0), p.n_layers - 1);
        }
      }
      // slot of this segment: sorted by start layer under layered transport, so that
      // the lanes of a wave read the same table rows and cross similar numbers of layers
      const int slot = wbase + (kLayers ? (int)wave_rank<8>(key) : lane);
      wave_fence();  // the previous tile's slots have been read
      s_q0[slot] = q0;
      s_q1[slot] = q1;
      s_q2[slot] = q2;
      s_q3[slot] = q3;
      s_fl01[slot] = fl_n.y;
      if constexpr (!kLayers) s_dx[slot] = make_float2(dXs, inv_q);
      if constexpr (kRecords) {
        s_rec[slot] = make_ulonglong2(id, i < p.n ? (unsigned long long)p.rec_off[i] : 0ull);
        s_nch[slot] = n_ch;
      }
      // ---- 2. record numbers: lane L holds slot L's counts and, below, offsets
      if constexpr (kLayers) {
        const int to = (slot - wbase) << 2;
        n_ch = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)n_ch);
        n_fl = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)n_fl);
        if (p.n_showers > 1) sh_of = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)sh_of);
      }
      if constexpr (MODE == MODE_PROPAGATE) {
        if (share == 0) {
          const uint32_t v_in = (uint32_t)__popcll(__ballot(i < p.n)), v_skip = (uint32_t)__popcll(__ballot(status == 2)),
                         v_below = (uint32_t)__popcll(__ballot(status == 1));
          const uint32_t v_fl = (p.emission & CPHOT_EMIT_FLUORESCENCE) ? wave_total(n_fl) : 0u;
          const uint32_t v_cut = (p.cuts & CPHOT_CUT_TRACK) ? wave_total(cut1) : 0u;
          if (lane == 0) {
            atomicAdd(&s_cnt[CPHOT_C_SEGMENTS_IN], (unsigned long long)v_in);
            if (v_skip) atomicAdd(&s_cnt[CPHOT_C_SEGMENTS_SKIPPED], (unsigned long long)v_skip);
            if (v_below) atomicAdd(&s_cnt[CPHOT_C_SEGMENTS_BELOW_THRESHOLD], (unsigned long long)v_below);
            if (v_fl) atomicAdd(&s_cnt[CPHOT_C_RECORDS_FLUORESCENCE], (unsigned long long)v_fl);
            if (v_cut) atomicAdd(&s_cnt[CPHOT_C_RECORDS_CULLED_TRACK], (unsigned long long)v_cut);
          }
        }
      }
      wave_fence();  // the slots are complete
      // A tile's records are numbered shower by shower (nearly always one), so that the
      // shower is the same in every lane and takes no slot memory.
      const uint32_t all_ch = n_ch, all_fl = n_fl;
      for (uint64_t todo = __ballot((all_ch | all_fl) != 0u); todo;) {
        ShowerState S;
        S.sh = 0;
        if (p.n_showers > 1) S.sh = __builtin_amdgcn_readlane((int)sh_of, (int)__builtin_ctzll(todo));
        const bool mine = p.n_showers <= 1 || (int)sh_of == S.sh;
        todo &= ~__ballot(mine);
        n_ch = mine ? all_ch : 0u;
        n_fl = mine ? all_fl : 0u;
        const uint32_t end_ch = wave_scan_add(n_ch), end_fl = wave_scan_add(n_fl);
        const uint32_t total_ch = (uint32_t)__builtin_amdgcn_readlane((int)end_ch, 63);
        const uint32_t total_fl = (uint32_t)__builtin_amdgcn_readlane((int)end_fl, 63);
        // ---- 3. rounds of 64 records, Cherenkov rounds first (at most 2^22, 2^5 shares). In a
        // tile of several showers the shares go round with the shower, so that showers of a
        // round or two are spread over its units (100 showers of a segment each 112 -> 36 us,
        // through the network 253 -> 71). A tile of one shower is not turned: the same share of
        // every tile then has the longer end (100 curved showers of 64 segments 82 -> 66 us).
        const uint32_t rounds_ch = (total_ch + 63) >> 6, rounds = rounds_ch + ((total_fl + 63) >> 6);
        uint32_t part = share;
        if (p.n_showers > 1 && __ballot((all_ch | all_fl) != 0u && !mine))
          part = (share + ((uint32_t)S.sh << (sub - p.sub_shift))) & ((1u << sub) - 1u);
        const uint32_t r_first = rounds * part >> sub, r_end = rounds * (part + 1) >> sub;
        if (r_first == r_end) continue;
        {
          const double* g = p.geom + 5 * (int64_t)S.sh;
          S.core_x = uniform((float)g[0]);
          S.core_y = uniform((float)g[1]);
          S.x0 = uniform(S.core_x - p.half_x);
          S.y0 = uniform(S.core_y - p.half_y);
          S.x64 = uniform((double)S.core_x - p.half_x64);
          S.y64 = uniform((double)S.core_y - p.half_y64);
          S.axx = S.axy = S.axz = 0.f;
          if constexpr (kTime) {
            S.axx = uniform((float)g[2]);
            S.axy = uniform((float)g[3]);
            S.axz = uniform((float)g[4]);
          }
        }
        // Window counts stay below 2^32: a block whose units of one shower could take them beyond
        // 2^31 leaves its window for the global bins, until the next shower. A CU needs some ten
        // seconds for that many records.
        bool use_win = n_hist != 0 && S.sh == win_sh;
        if (use_win) {
          unsigned long long sum = ((total_ch + total_fl) >> sub) + 192u;  // no unit of the tile has more
          if (lane == 0) sum += atomicAdd(&s_since, sum);
          use_win = !__builtin_amdgcn_readfirstlane((int)(sum > (1ull << 31)));
        }
        uint32_t done = 0, culled = 0, fallback = 0, not_emitted = 0;  // the same in every lane
        uint32_t packed = 0, in_packed = 0;  // this lane's counts of states 0..3, 8 bits each; additions since the last unpacking
        auto unpack = [&]() {
          const uint32_t a = wave_total(packed & 0x00ff00ffu), b = wave_total((packed >> 8) & 0x00ff00ffu);
          if (lane == 0) {
            atomicAdd(&s_cnt[CPHOT_C_RECORDS_BINNED], (unsigned long long)(a & 0xffffu));
            atomicAdd(&s_cnt[CPHOT_C_RECORDS_ABSORBED], (unsigned long long)(a >> 16));
            atomicAdd(&s_cnt[CPHOT_C_RECORDS_UPWARD], (unsigned long long)(b & 0xffffu));
            atomicAdd(&s_cnt[CPHOT_C_RECORDS_OUTSIDE], (unsigned long long)(b >> 16));
          }
          packed = 0;
          in_packed = 0;
        };
        auto load_slot = [&](int s, SegState& g) {
          g.q0 = s_q0[s];
          g.q1 = s_q1[s];
          g.q2 = s_q2[s];
          g.q3 = s_q3[s];
          g.fl01 = s_fl01[s];
          g.dX = 0.f;
          g.inv_q = g.q2.w;
          if constexpr (!kLayers) {
            const float2 x = s_dx[s];
            g.dX = x.x;
            g.inv_q = x.y;
          }
        };
        // one record: counters and bins
        auto consume = [&](const KParams& p, const Photon& ph) {
          if (!EXT || ph.state != kStateNotEmitted) packed += 1u << ph.state;
          if (ph.state == 0u) {
            if constexpr (DETECTOR == CPHOT_DETECTOR_GRID) {
              const int lx = ph.ix - win.x0, ly = ph.iy - win.y0;
              if (use_win && (unsigned)lx < (unsigned)win.w && (unsigned)ly < (unsigned)win.h)
                atomicAdd(&s_hist[ly * win.w + lx], 1u);
              else
                add_bin(p, (int64_t)S.sh * p.nx * p.ny + ph.bin, p.bunch);
            } else {
              const int64_t nsph = (int64_t)H.snx * H.sny;
              const int64_t gb = (int64_t)S.sh * nsph + ph.bin;
              if (use_win) atomicAdd(&s_hist[ph.bin], 1u);
              else add_bin(p, gb, p.bunch);
              if (H.n_t > 0) {
                if (use_win && ph.tbin < H.hist_tw) atomicAdd(&s_hist[nsph + ph.bin * H.hist_tw + ph.tbin], 1u);
                else atomicAdd(p.thist + gb * (H.n_t + 1) + ph.tbin, p.bunch);
              }
            }
          }
        };
        // list mode, called by all lanes of the wave: rows of 64 bytes, gathered in LDS so
        // that four lanes store a row and one instruction 16 of them, past the caches. Bound
        // by the stores: 3.5e6 records 101 us with 16 bytes from each lane, 64 apart, 61 us
        // gathered and 53 us non-temporal (4.2 TB/s).
        auto write_rows = [&](const KParams& p, const Photon& ph, int s, bool fl, uint32_t kk, bool live) {
          const ulonglong2 rec = s_rec[s];
          const uint32_t k = fl ? kk + s_nch[s] : kk;
          int64_t at = (int64_t)rec.y + (int64_t)k;
          if (!live || at >= p.rec_cap) at = -1;
          const uint4 part[4] = {
              make_uint4((uint32_t)rec.x, (uint32_t)(rec.x >> 32), k, ph.state >> 3),
              make_uint4((uint32_t)ph.bin, (uint32_t)ph.tbin, __float_as_uint(ph.x), __float_as_uint(ph.y)),
              make_uint4(__float_as_uint(ph.z), __float_as_uint(ph.t), __float_as_uint(ph.tau), __float_as_uint(ph.lam)),
              make_uint4(__float_as_uint(ph.ux), __float_as_uint(ph.uy), __float_as_uint(ph.uz),
                         __float_as_uint(ph.u3 * kU24))};
          uint4* rows = s_row + (wbase >> 6) * (4 * kRowsAtOnce);
#pragma unroll
          for (int h = 0; h < 64 / kRowsAtOnce; ++h) {
            wave_fence();  // the rows before these have been read
            if (lane / kRowsAtOnce == h) {
#pragma unroll
              for (int q = 0; q < 4; ++q) rows[4 * (lane % kRowsAtOnce) + (q ^ (lane >> 1 & 3))] = part[q];
            }
            wave_fence();
#pragma unroll
            for (int q = 0; q < kRowsAtOnce / 16; ++q) {
              const int row = 16 * q + (lane >> 2), of = kRowsAtOnce * h + row;
              const int64_t to = ((int64_t)__shfl((int)(at >> 32), of) << 32) | (uint32_t)__shfl((int)at, of);
              const uint4 v = rows[4 * row + ((lane & 3) ^ (row >> 1 & 3))];
              if (to >= 0) {
                typedef uint32_t part_t __attribute__((ext_vector_type(4), aligned(alignof(cphot_photon_record))));
                __builtin_nontemporal_store(part_t{v.x, v.y, v.z, v.w}, reinterpret_cast<part_t*>(p.rec + to) + (lane & 3));
              }
            }
          }
        };
        uint32_t q_len = 0;  // this wave's queue of deferred records (the same in every lane)
        uint32_t* queue = s_queue + (kDefer ? wbase : 0);
        uint32_t w_len = 0;  // the same of the second queue
        uint32_t* walks = s_queue + (kQueues == 2 ? BS + wbase : 0);
        for (uint32_t r = r_first; r < r_end; ++r) {
          const KParams& pr = fresh_params();
          const bool fl = r >= rounds_ch;
          const uint32_t j0 = (fl ? r - rounds_ch : r) << 6, total = fl ? total_fl : total_ch;
          const uint32_t cnt = fl ? n_fl : n_ch, off = (fl ? end_fl : end_ch) - cnt;
          // slot of record j0 + lane: the last slot that starts at or before it. The slots
          // that start inside the round push their number to the lane they start at (only
          // slots with records: no two at one lane); lane 0 gets the slot j0 lies in.
          const uint32_t cur = (uint32_t)__popcll(__ballot(off <= j0)) - 1u;
          const uint32_t d = off - j0;
          const bool starts = cnt != 0u && d - 1u < 63u;
          uint32_t at = (uint32_t)__builtin_amdgcn_ds_permute(starts ? (int)(d << 2) : 0, lane);
          at = wave_scan_max(lane == 0 ? cur : at);
          const uint32_t kk = j0 + (uint32_t)lane - (uint32_t)__builtin_amdgcn_ds_bpermute((int)(at << 2), (int)off);
          const bool valid = j0 + (uint32_t)lane < total;
          const int s = wbase + (int)at;
          done += min(total - j0, 64u);
          Photon ph;
          ph.state = kStateNotEmitted;
          ph.culled = 0;
          if (kMlp || valid) {
            SegState g;
            load_slot(s, g);
            trace<TRANSPORT, DETECTOR, kTime, kRecords, EXT>(H, pr, T, g, S, fl, kk, valid, ph);
            if (!kRecords && valid && (!kDefer || ph.state != kStateDeferred)) consume(pr, ph);
          }
          if constexpr (kRecords) write_rows(pr, ph, s, fl, kk, valid && (!kDefer || ph.state != kStateDeferred));
          if constexpr (MODE == MODE_PROPAGATE) {
            if (H.cuts & CPHOT_CUT_PHOTON) culled += (uint32_t)__popcll(__ballot(valid && ph.culled));
            if (EXT) not_emitted += (uint32_t)__popcll(__ballot(valid && ph.state == kStateNotEmitted));
            if (++in_packed == 255u) unpack();
          }
          if constexpr (kDefer) {
            // wave-level compaction: deferred records take consecutive entries of this wave's
            // queue (ballot and prefix count of the lanes below); the wave traces the queue
            // exactly when they would not fit, and after the last round. Of the curved
            // network's and table's records some leave the closed-form sums too: these go to
            // a second queue in the same way, so that no wave runs the sums and the much
            // longer shell walk for the same 64 records (of the inclined shower's 12 % outside
            // the table 4 in 10 are walked: 1.36 ms with one queue, 1.15 with two; network
            // 2.29 and 2.04 ms).
            const bool push = valid && ph.state == kStateDeferred, last = r + 1u == r_end;
            const uint32_t n_push = (uint32_t)__popcll(__ballot(push));
            auto append = [&](uint32_t* q, uint32_t& len, bool take, uint32_t e) {
              const uint64_t mask = __ballot(take);
              if (take)
                q[len + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u))] = e;
              len += (uint32_t)__popcll(mask);
            };
            // traces the queue's records; true in a lane whose record e is deferred again
            auto drain = [&](auto transport, const uint32_t* q, uint32_t& len, uint32_t& e) {
              wave_fence();  // the queue's entries are complete
              const KParams& pq = fresh_params();
              const bool mine = (uint32_t)lane < len;
              e = mine ? q[lane] : 0u;
              const int qs = wbase + (int)(e & 63u);
              const bool qfl = (e & 64u) != 0u;
              const uint32_t qk = e >> 7;
              Photon pe;
              pe.state = kStateDeferred;
              if (mine) {
                SegState g;
                load_slot(qs, g);
                trace<decltype(transport)::value, DETECTOR, kTime, kRecords, EXT>(pq, pq, T, g, S, qfl, qk, true, pe);
              }
              const bool done_with = pe.state != kStateDeferred;
              if constexpr (kRecords) write_rows(pq, pe, qs, qfl, qk, done_with);
              else if (done_with) consume(pq, pe);
              wave_fence();  // every lane has read its entry before the queue takes new ones
              len = 0;
              if constexpr (MODE == MODE_PROPAGATE) {
                if (++in_packed == 255u) unpack();
              }
              return mine && !done_with;
            };
            // pass 0 makes room for the round's entries; the others empty the queues after
            // the last round
#pragma unroll 1
            for (int pass = 0; pass < (last ? 1 + kQueues : 1); ++pass) {
              bool again = false;
              uint32_t e = 0, e_walk;
              if (pass == 0 ? q_len + n_push > 64u : pass == 1 && q_len > 0u) {
                fallback += q_len;
                again = drain(std::integral_constant<int, kExact>{}, queue, q_len, e);
              }
              if constexpr (kQueues == 2) {
                if (pass < 2 ? w_len + (uint32_t)__popcll(__ballot(again)) > 64u : w_len > 0u)
                  drain(std::integral_constant<int, kTransportCurvedWalk>{}, walks, w_len, e_walk);
                append(walks, w_len, again, e);
              }
              if (pass == 0) append(queue, q_len, push, at | (fl ? 64u : 0u) | (kk << 7));
            }
          }
        }
        if constexpr (MODE == MODE_PROPAGATE) {
          unpack();
          if (lane == 0) {
            if (done) atomicAdd(&s_cnt[CPHOT_C_RECORDS_GENERATED], (unsigned long long)done);
            if (fallback) atomicAdd(&s_cnt[CPHOT_C_SURROGATE_FALLBACK], (unsigned long long)fallback);
            if (culled) atomicAdd(&s_cnt[CPHOT_C_RECORDS_CULLED_PHOTON], (unsigned long long)culled);
            if (not_emitted) atomicAdd(&s_cnt[CPHOT_C_RECORDS_NOT_EMITTED], (unsigned long long)not_emitted);
          }
        }
      }
    }
  }
  if constexpr (MODE == MODE_PROPAGATE) {
    __syncthreads();
    if (win_sh >= 0) flush_window<BS, DETECTOR>(p, s_hist, win, win_sh);
    if (p.counters && tid < CPHOT_NCOUNTERS) {
      // one global atomic per counter and block (same-address device atomics
      // serialise, so their number must stay small)
      const unsigned long long v =
          tid == CPHOT_C_PHOTONS_BINNED ? s_cnt[CPHOT_C_RECORDS_BINNED] * p.bunch : s_cnt[tid];
      if (v) atomicAdd(p.counters + tid, v);
    }
  }
}

#if CPHOT_BLOCK == 256
// Records and expected records per segment.
template <bool EXT>
__global__ __launch_bounds__(256) void k_counts(KParams p) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < p.n; i += (int64_t)gridDim.x * 256) {
    const uint64_t id = p.first_id + (uint64_t)i * p.id_stride;
    const SegResult r = segment_setup<EXT>(p, p.x0[i], p.y0[i], p.z0[i], p.x1[i], p.y1[i], p.z1[i], p.beta[i],
                                           p.charge[i], p.dedx ? p.dedx[i] : 0.0f, id);
    p.counts[i] = r.n + r.nf[0] + r.nf[1] + r.nf[2];
    if (p.expected) p.expected[i] = r.status == 0 ? r.mu : 0.0;
  }
}
#endif

namespace {

template <int BS, int T, int D, int M, bool EXT>
hipError_t launch_one(const KParams& p, dim3 grid, size_t lds, hipStream_t s) {
  hipLaunchKernelGGL((k_propagate<BS, T, D, M, EXT>), grid, dim3(BS), lds, s, p);
  return hipGetLastError();
}

#if CPHOT_BLOCK != 1024
template <int BS, int T, int D>
hipError_t launch_mode(const KParams& p, int mode, dim3 grid, size_t lds, hipStream_t s) {
  const bool ext = p.poisson || p.spectrum == CPHOT_SPECTRUM_DISPERSIVE;
  if (mode == MODE_PROPAGATE)
    return ext ? launch_one<BS, T, D, MODE_PROPAGATE, true>(p, grid, lds, s)
               : launch_one<BS, T, D, MODE_PROPAGATE, false>(p, grid, lds, s);
  return ext ? launch_one<BS, T, D, MODE_RECORDS, true>(p, grid, lds, s)
             : launch_one<BS, T, D, MODE_RECORDS, false>(p, grid, lds, s);
}
#endif

template <int BS, int T, int D>
KernelInfo info_one() {
  hipFuncAttributes a;
  // the EXT kernels declare the same static LDS and run at the same waves per SIMD
  if (hipFuncGetAttributes(&a, reinterpret_cast<const void*>(&k_propagate<BS, T, D, MODE_PROPAGATE, false>)) != hipSuccess)
    return {0, 1};
  const int regs = (std::max(a.numRegs, 1) + 7) / 8 * 8;  // allocated by eights from 512 per lane and SIMD
  return {a.sharedSizeBytes, std::min(8, 512 / regs)};
}

}  // namespace

// Each block size is compiled by itself (CPHOT_BLOCK), so that they build side by side.
// The large size serves the library's own choice: 1024 threads, or 768
// for the network kernels, whose registers allow three waves per SIMD.
#if CPHOT_BLOCK == 1024
template <int T>
constexpr int kBig = kMlpTransport<T> ? 768 : 1024;

template <>
hipError_t launch_block<1024>(const KParams& p, int mode, dim3 grid, size_t lds, hipStream_t s) {
  (void)mode;
  const bool ext = p.poisson || p.spectrum == CPHOT_SPECTRUM_DISPERSIVE;
#define CPHOT_BIG(T, D) \
  return ext ? launch_one<kBig<T>, T, D, MODE_PROPAGATE, true>(p, grid, lds, s) \
             : launch_one<kBig<T>, T, D, MODE_PROPAGATE, false>(p, grid, lds, s);
  if (p.detector == CPHOT_DETECTOR_SPHERES) switch (p.transport) {
    case CPHOT_TRANSPORT_STRAIGHT: CPHOT_BIG(CPHOT_TRANSPORT_STRAIGHT, 1)
    case CPHOT_TRANSPORT_LAYERED: CPHOT_BIG(CPHOT_TRANSPORT_LAYERED, 1)
    case CPHOT_TRANSPORT_SURROGATE: CPHOT_BIG(CPHOT_TRANSPORT_SURROGATE, 1)
    case CPHOT_TRANSPORT_TABLE: CPHOT_BIG(CPHOT_TRANSPORT_TABLE, 1)
    default: return hipErrorInvalidValue;
  }
  switch (p.transport) {
    case CPHOT_TRANSPORT_STRAIGHT: CPHOT_BIG(CPHOT_TRANSPORT_STRAIGHT, 0)
    case CPHOT_TRANSPORT_LAYERED: CPHOT_BIG(CPHOT_TRANSPORT_LAYERED, 0)
    case CPHOT_TRANSPORT_SURROGATE: CPHOT_BIG(CPHOT_TRANSPORT_SURROGATE, 0)
    case CPHOT_TRANSPORT_CURVED: CPHOT_BIG(CPHOT_TRANSPORT_CURVED, 0)
    case CPHOT_TRANSPORT_TABLE: CPHOT_BIG(CPHOT_TRANSPORT_TABLE, 0)
    case kTransportCurvedWalk: CPHOT_BIG(kTransportCurvedWalk, 0)
    case kTransportCurvedTable: CPHOT_BIG(kTransportCurvedTable, 0)
    case kTransportCurvedSurrogate: CPHOT_BIG(kTransportCurvedSurrogate, 0)
    default: return hipErrorInvalidValue;
  }
#undef CPHOT_BIG
}

template <>
KernelInfo info_block<1024>(const KParams& p) {
  if (p.detector == CPHOT_DETECTOR_SPHERES) switch (p.transport) {
    case CPHOT_TRANSPORT_STRAIGHT: return info_one<1024, CPHOT_TRANSPORT_STRAIGHT, 1>();
    case CPHOT_TRANSPORT_LAYERED: return info_one<1024, CPHOT_TRANSPORT_LAYERED, 1>();
    case CPHOT_TRANSPORT_TABLE: return info_one<1024, CPHOT_TRANSPORT_TABLE, 1>();
    default: return info_one<768, CPHOT_TRANSPORT_SURROGATE, 1>();
  }
  switch (p.transport) {
    case CPHOT_TRANSPORT_STRAIGHT: return info_one<1024, CPHOT_TRANSPORT_STRAIGHT, 0>();
    case CPHOT_TRANSPORT_LAYERED: return info_one<1024, CPHOT_TRANSPORT_LAYERED, 0>();
    case CPHOT_TRANSPORT_SURROGATE: return info_one<768, CPHOT_TRANSPORT_SURROGATE, 0>();
    case CPHOT_TRANSPORT_CURVED: return info_one<1024, CPHOT_TRANSPORT_CURVED, 0>();
    case CPHOT_TRANSPORT_TABLE: return info_one<1024, CPHOT_TRANSPORT_TABLE, 0>();
    case kTransportCurvedWalk: return info_one<1024, kTransportCurvedWalk, 0>();
    case kTransportCurvedTable: return info_one<1024, kTransportCurvedTable, 0>();
    default: return info_one<768, kTransportCurvedSurrogate, 0>();
  }
}
#else
template <>
hipError_t launch_block<CPHOT_BLOCK>(const KParams& p, int mode, dim3 grid, size_t lds, hipStream_t s) {
  constexpr int BS = CPHOT_BLOCK;
  const bool g = p.detector == CPHOT_DETECTOR_GRID;
  switch (p.transport) {
    case CPHOT_TRANSPORT_STRAIGHT: return g ? launch_mode<BS, 0, 0>(p, mode, grid, lds, s) : launch_mode<BS, 0, 1>(p, mode, grid, lds, s);
    case CPHOT_TRANSPORT_LAYERED: return g ? launch_mode<BS, 1, 0>(p, mode, grid, lds, s) : launch_mode<BS, 1, 1>(p, mode, grid, lds, s);
    case CPHOT_TRANSPORT_SURROGATE: return g ? launch_mode<BS, 2, 0>(p, mode, grid, lds, s) : launch_mode<BS, 2, 1>(p, mode, grid, lds, s);
    case CPHOT_TRANSPORT_CURVED: return launch_mode<BS, 3, 0>(p, mode, grid, lds, s);  // grid detector only
    case kTransportCurvedWalk: return launch_mode<BS, kTransportCurvedWalk, 0>(p, mode, grid, lds, s);
    case CPHOT_TRANSPORT_TABLE: return g ? launch_mode<BS, 4, 0>(p, mode, grid, lds, s) : launch_mode<BS, 4, 1>(p, mode, grid, lds, s);
    case kTransportCurvedTable: return launch_mode<BS, kTransportCurvedTable, 0>(p, mode, grid, lds, s);
    default: return launch_mode<BS, kTransportCurvedSurrogate, 0>(p, mode, grid, lds, s);
  }
}

template <>
KernelInfo info_block<CPHOT_BLOCK>(const KParams& p) {
  constexpr int BS = CPHOT_BLOCK;
  const bool g = p.detector == CPHOT_DETECTOR_GRID;
  switch (p.transport) {
    case CPHOT_TRANSPORT_STRAIGHT: return g ? info_one<BS, 0, 0>() : info_one<BS, 0, 1>();
    case CPHOT_TRANSPORT_LAYERED: return g ? info_one<BS, 1, 0>() : info_one<BS, 1, 1>();
    case CPHOT_TRANSPORT_SURROGATE: return g ? info_one<BS, 2, 0>() : info_one<BS, 2, 1>();
    case CPHOT_TRANSPORT_CURVED: return info_one<BS, 3, 0>();
    case kTransportCurvedWalk: return info_one<BS, kTransportCurvedWalk, 0>();
    case CPHOT_TRANSPORT_TABLE: return g ? info_one<BS, 4, 0>() : info_one<BS, 4, 1>();
    case kTransportCurvedTable: return info_one<BS, kTransportCurvedTable, 0>();
    default: return info_one<BS, kTransportCurvedSurrogate, 0>();
  }
}
#endif

#if CPHOT_BLOCK == 256
KernelInfo propagate_info(const KParams& p, int block_size) {
  switch (block_size) {
    case 128: return info_block<128>(p);
    case 512: return info_block<512>(p);
    case kBigBlock: return info_block<1024>(p);
    default: return info_block<256>(p);
  }
}

hipError_t launch_propagate(const KParams& p, int mode, int block_size, int grid_blocks, size_t lds_bytes,
                            hipStream_t stream) {
  if (mode == MODE_COUNTS) {
    if (p.poisson || p.spectrum == CPHOT_SPECTRUM_DISPERSIVE)
      hipLaunchKernelGGL(k_counts<true>, dim3(grid_blocks), dim3(256), 0, stream, p);
    else
      hipLaunchKernelGGL(k_counts<false>, dim3(grid_blocks), dim3(256), 0, stream, p);
    return hipGetLastError();
  }
  const dim3 grid(grid_blocks);
  switch (block_size) {
    case 128: return launch_block<128>(p, mode, grid, lds_bytes, stream);
    case 512: return launch_block<512>(p, mode, grid, lds_bytes, stream);
    case kBigBlock: return launch_block<1024>(p, mode, grid, lds_bytes, stream);
    default: return launch_block<256>(p, mode, grid, lds_bytes, stream);
  }
}
#endif

}  // namespace cphot
