// Exact walks of one photon in FP64, for tabulated corrections and training
// targets (not the propagation hot path, which walks in FP32). Both follow the
// same laws as the FP32 walks of cphot_device.h, carried in double so that the
// stored corrections are limited by the physics rather than by rounding.
// Layer data: lay[i] = (n - 1, 1/n, Rayleigh part, aerosol part) as float4;
// the optical depth is returned split into its Rayleigh and aerosol path
// integrals, sum R_i l_i and sum A_i l_i, so that tau = sp.x tR + sp.y tA for a
// wavelength with spectral factors sp.
#pragma once

#include <hip/hip_runtime.h>

namespace cphot {

struct Walk64 {
  double across;  // planar: horizontal travel along the azimuth; curved: central angle swept
  double len;     // geometric path length
  double opt;     // sum (n - 1) l
  double tR, tA;  // Rayleigh and aerosol path integrals
};

// Planar layers (Sec. 3.4.2): from height h0 with cos of the zenith angle c0
// (downward) to the observation level h_obs. Snell's law conserves the
// horizontal part of n u: in layer i the sine is s0 (1 - e_i), e_i =
// (d_i - d_0) / (1 + d_i), and the squared cosine c0^2 + s0^2 e_i (2 - e_i).
// The start layer is `i0` (its top boundary counts as inside it), or the layer
// containing h0 when i0 < 0.
__device__ inline void planar_walk_f64(const float4* __restrict__ lay, double dh, int n_layers, double h_obs,
                                       double h0, double c0, Walk64& w, int i0 = -1) {
  const double s0 = sqrt((1.0 - c0) * (1.0 + c0));
  int i = i0 >= 0 ? i0 : min((int)(h0 / dh), n_layers - 1);
  const int obs = (int)floor(h_obs / dh);
  const double d0 = (double)lay[i].x;
  w.across = w.len = w.opt = w.tR = w.tA = 0.0;
  double z = h0;
  for (;;) {
    const float4 L = lay[i];
    const double di = (double)L.x;
    const double e = (di - d0) / (1.0 + di);
    const double s = s0 * (1.0 - e);
    const double c = sqrt(c0 * c0 + s0 * s0 * e * (2.0 - e));
    const double zb = (i > obs) ? i * dh : h_obs;
    const double path = (z - zb) / c;
    w.across += path * s;
    w.len += path;
    w.opt += di * path;
    w.tR += (double)L.z * path;
    w.tA += (double)L.w * path;
    if (i <= obs) break;
    z = zb;
    --i;
  }
}

// Spherical shells of a curved Earth (Sec. 3.3.4): the impact-parameter deficit
// D = (R + h) - p = (h - h0) + (R + h0) [(1 - s0) - s0 (d0 - d_i) / (1 + d_i)]
// is carried without radius-sized subtractions; a chord from ha down to hb is
// (ha - hb)(2R + ha + hb) / (ra ca + rb cb) and sweeps asin(p l / (ra rb)); a ray
// turns round inside a shell where D would become negative and is totally
// reflected where the next shell's D is not positive. Start at height h0 with
// local zenith cosine c0 (downward), in shell i0 (or the shell containing h0 when
// i0 < 0). Returns false if the ray does not reach the sphere R + h_obs.
__device__ inline bool shell_walk_f64(const float4* __restrict__ lay, double dh, int n_layers, double h_obs,
                                      double Re, double h0, double c0, Walk64& w, int i0 = -1) {
  const double s0 = sqrt((1.0 - c0) * (1.0 + c0));
  int i = i0 >= 0 ? i0 : min((int)(h0 / dh), n_layers - 1);
  const int obs = (int)floor(h_obs / dh);
  const double A = Re + h0;
  const double c1 = c0 * c0 / (1.0 + s0);
  const double d0 = (double)lay[i].x;
  auto bracket = [&](int k) {
    const double dk = (double)lay[k].x;
    return c1 - s0 * (d0 - dk) / (1.0 + dk);
  };
  double h = h0;
  w.across = w.len = w.opt = w.tR = w.tA = 0.0;
  bool down = c0 > 0.0;
  for (int iter = 0; iter < 8 * n_layers; ++iter) {
    const double br = bracket(i);
    const double ra = Re + h;
    const double Da = A * br + (h - h0);
    const double rca = sqrt(fmax(Da * (2.0 * ra - Da), 0.0));
    const double pa = ra - Da;
    double ell, dpsi;
    bool to_top = false;
    if (down) {
      const double hb = (i == obs) ? h_obs : i * dh;
      const double Db = A * br + (hb - h0);
      if (Db > 0.0) {
        const double rb = Re + hb;
        const double rcb = sqrt(Db * (2.0 * rb - Db));
        ell = (h - hb) * (2.0 * Re + h + hb) / (rca + rcb);
        dpsi = asin(pa * ell / (ra * rb));
        h = hb;
      } else {
        const double ho = (i + 1) * dh;
        const double ro = Re + ho;
        const double Do = A * br + (ho - h0);
        const double rco = sqrt(fmax(Do * (2.0 * ro - Do), 0.0));
        ell = rca + rco;
        dpsi = atan2(rca, pa) + atan2(rco, pa);
        h = ho;
        down = false;
        to_top = true;
      }
    } else {
      const double ho = (i + 1) * dh;
      const double ro = Re + ho;
      const double Do = A * br + (ho - h0);
      const double rco = sqrt(fmax(Do * (2.0 * ro - Do), 0.0));
      ell = (ho - h) * (2.0 * Re + ho + h) / (rco + rca);
      dpsi = asin(pa * ell / (ra * ro));
      h = ho;
      to_top = true;
    }
    const float4 L = lay[i];
    w.len += ell;
    w.opt += (double)L.x * ell;
    w.tR += (double)L.z * ell;
    w.tA += (double)L.w * ell;
    w.across += dpsi;
    if (!to_top) {
      if (i == obs) return true;
      if (!(A * bracket(i - 1) + (h - h0) > 0.0)) {
        down = false;
        continue;
      }
      --i;
      continue;
    }
    if (i + 1 >= n_layers) return false;
    if (!(A * bracket(i + 1) + (h - h0) > 0.0)) {
      down = true;
      continue;
    }
    ++i;
  }
  return false;
}

// Reciprocal and square root of positive, normal doubles by Newton's iteration from the
// hardware's estimates, within two units in the last place (the walk's sums are rounded to
// FP32 afterwards).
__device__ __forceinline__ double rcp_f64(double a) {
  double y = __builtin_amdgcn_rcp(a);
  y = fma(fma(-a, y, 1.0), y, y);
  return fma(fma(-a, y, 1.0), y, y);
}
__device__ __forceinline__ double sqrt_f64(double a) {
  const double y = __builtin_amdgcn_rsq(a);
  double g = a * y, h = 0.5 * y;
  double r = fma(-h, g, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  r = fma(-g, g, a);
  return fma(r, h, g);
}

// The sums of shell_walk_f64 for a ray that goes straight down through every shell, as
// nearly all do (nd[i] = n - 1 and 1 / n of shell i): one reciprocal and two square roots a
// shell where the general walk takes divisions, and the arc sine of the small angle of a
// shell by its series (x <= 0.01: the omitted term is below 4e-18 of it). The number of
// shells is known beforehand; false, and the sums void, where the ray turns or is reflected
// in one of them.
__device__ inline bool shell_descent_f64(const double2* __restrict__ nd, const float4* __restrict__ lay, double dh,
                                         int n_layers, double h_obs, double Re, double h0, double c0, Walk64& w) {
  const double s0 = sqrt_f64(fmax((1.0 - c0) * (1.0 + c0), 1e-200));
  int i = min((int)(h0 / dh), n_layers - 1);
  const int obs = (int)floor(h_obs / dh);
  const double A = Re + h0, As0 = A * s0;
  const double Ac1 = A * (c0 * c0 / (1.0 + s0));
  const double d0 = nd[i].x;
  w.across = w.len = w.opt = w.tR = w.tA = 0.0;
  if (!(c0 > 0.0) || i < obs) return false;
  bool down = true;
  double ra = A, ha = 0.0;  // ha, hb: heights relative to the start
  auto shell = [&](int k, double hb_abs) {
    const double2 n = nd[k];
    const float4 L = lay[k];
    const double br = fma(As0 * (n.x - d0), n.y, Ac1);
    const double rb = Re + hb_abs, hb = hb_abs - h0;
    const double Da = br + ha, Db = br + hb;
    const double rca = sqrt_f64(fmax(Da * fma(2.0, ra, -Da), 1e-200)), rcb = sqrt_f64(Db * fma(2.0, rb, -Db));
    const double rr = ra * rb;
    const double q = (ha - hb) * (ra + rb) * rcp_f64((rca + rcb) * rr);
    const double ell = q * rr, x = (ra - Da) * q, x2 = x * x;
    down = down && Da >= 0.0 && Db > 0.0 && x < 0.01;
    w.across += fma(x * x2, fma(x2, fma(x2, 15.0 / 336.0, 3.0 / 40.0), 1.0 / 6.0), x);
    w.len += ell;
    w.opt = fma(n.x, ell, w.opt);
    w.tR = fma((double)L.z, ell, w.tR);
    w.tA = fma((double)L.w, ell, w.tA);
    ha = hb;
    ra = rb;
  };
#pragma unroll 2
  for (; i > obs; --i) shell(i, i * dh);
  shell(obs, h_obs);
  return down;
}

// Straight chord from height h0 at local zenith cosine c0 to the sphere R + h_obs,
// cancellation-free root, and the central angle it sweeps.
__device__ inline void chord_f64(double Re, double h_obs, double h0, double c0, double& len, double& psi) {
  const double r0 = Re + h0, r1 = Re + h_obs, s0 = sqrt((1.0 - c0) * (1.0 + c0));
  const double drs = (h0 - h_obs) * (r0 + r1);
  len = drs / (r0 * c0 + sqrt(r0 * r0 * c0 * c0 - drs));
  psi = asin(len * s0 / r1);
}

}  // namespace cphot
