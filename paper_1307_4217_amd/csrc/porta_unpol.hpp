// Sweep kernel of the unpolarized problem (Stokes I only): the scalar form of
// Eqs. fsint / fsbez with K' = 0 and the emission eps^0_0, which PORTA also solves
// (the non-LTE problem of unpolarized radiation, Sect. 1).  Same plane walk, thread
// mapping, control points and fused J reduction as k_sweep_plane; the plane state
// holds one value per node and frequency ([ray][frequency][node]).
#pragma once

#include "porta_kernels.hpp"

namespace porta {

template <class T>
__global__ void __launch_bounds__(256) k_sweep_plane_i(const PlaneArgs<T> a) {
  extern __shared__ double s_tab[];
  if ((int)blockIdx.x >= a.nstep) {
    jblock<1>(a, s_tab);
    return;
  }
  const StepBlock sb = step_block(a);
  const HemiArgs<T> h = hemi_args(a, sb.hemi);
  const int f0 = sb.chunk * a.fchunk, nf = min(a.fchunk, a.nfreq - f0);
  double* s_wn = s_tab;
  T* s_phi = reinterpret_cast<T*>(s_tab + a.fchunk);
  for (int t = threadIdx.x; t < nf; t += blockDim.x) {
    s_wn[t] = a.wn[f0 + t];
    s_phi[t] = a.phi[f0 + t];
  }
  __syncthreads();
  const int p = sb.bx * blockDim.x + threadIdx.x;
  if (p >= a.np) return;   // no barrier follows
  // M on the upwind plane, O, and P on the downwind plane (bilinear in the plane)
  const int ray = h.ray0 + sb.rb;
  const int j = p / a.nx, i = p - j * a.nx;
  const RayGeom& gM = layer_geom(a.geom, ray, a.nz, h.kO, h.kM, 0);
  const Stencil sM = make_stencil(i, j, a.nx, a.ny, gM);
  const size_t bM = (size_t)h.kM * a.np, bO = (size_t)h.kO * a.np + p;
  const double kapM = bil(a.kappa + bM, sM), kapO = (double)a.kappa[bO];
  const double SM = bil(a.emis + bM, sM) / kapM, SO = (double)a.emis[bO] / kapO;
  const double tau0M = 0.5 * (kapM + kapO) * gM.ds;
  double cM = 0.5 * (SM + SO), lamfac = 0.5;   // no downwind plane: linear control point
  if (h.kP >= 0) {
    const RayGeom& gP = layer_geom(a.geom, ray, a.nz, h.kO, h.kP, 1);
    const Stencil sP = make_stencil(i, j, a.nx, a.ny, gP);
    const size_t bP = (size_t)h.kP * a.np;
    const double kapP = bil(a.kappa + bP, sP);
    const double SP = bil(a.emis + bP, sP) / kapP;
    const double r = tau0M / (0.5 * (kapO + kapP) * gP.ds), inv = 0.5 / (1.0 + r), ir = 1.0 / r;
    const bool par = a.parabolic != 0;
    cM = control_cm(SM, SO, SP, SP - SO, r, inv, ir, par);
    lamfac = par ? control_cm(0.0, 1.0, 0.0, -1.0, r, inv, ir, true) : 1.0;   // unit source at O
  }
  StepSource<T> src;
  step_source(SM, SO, cM, src);
  const T tau0 = (T)tau0M, lf = (T)lamfac;
  const T w00 = (T)sM.w00, w10 = (T)sM.w10, w01 = (T)sM.w01, w11 = (T)sM.w11;

  const size_t fstride = (size_t)a.np;
  const size_t foff = ((size_t)sb.rb * a.nfreq + f0) * fstride;
  const T* ip = h.iprev ? h.iprev + foff : nullptr;
  T* op = h.inext + foff + p;
  double jacc = 0.0, lacc = 0.0;
  // one update (the scalar Eq. fsbez) at frequency f0 + f from the upwind intensity IM
  auto update = [&](int f, T IM) __attribute__((always_inline)) {
    const Coefs<T> cf = coefficients(tau0 * s_phi[f]);
    const StepSource<T> w = source_weights(cf);
    const T x = fma_t(w.c, src.c, dot3(w.a, src.a, cf.e, IM, w.b, src.b));
    __builtin_nontemporal_store(x, op + (size_t)f * fstride);   // as store4_nt
    const double W = s_wn[f];
    jacc = fma_t(W, (double)x, jacc);
    lacc = fma_t(W, (double)lambda_star(cf, lf), lacc);
  };
  if (!ip) {
    // the upwind plane is the boundary
    for (int f = 0; f < nf; ++f) update(f, h.ibound);
  } else {
    // the four corners of frequency f + 1 are loaded during the arithmetic of frequency f
    auto load = [&](int f, T v[4]) __attribute__((always_inline)) {
      const T* q = ip + (size_t)f * fstride;
      v[0] = q[sM.i00];
      v[1] = q[sM.i10];
      v[2] = q[sM.i01];
      v[3] = q[sM.i11];
    };
    // (never skipped, as in k_sweep_plane)
    T vA[4], vB[4];
    load(0, vA);
    int f = 0;
    for (; f + 1 < nf; f += 2) {
      load(f + 1, vB);
      update(f, bilinear(w10, w00, w01, w11, vA[1], vA[0], vA[2], vA[3]));
      load(min(f + 2, nf - 1), vA);
      update(f + 1, bilinear(w10, w00, w01, w11, vB[1], vB[0], vB[2], vB[3]));
    }
    if (f < nf) update(f, bilinear(w10, w00, w01, w11, vA[1], vA[0], vA[2], vA[3]));
  }
  if (h.jpart) {
    double* jp = h.jpart + ((size_t)sb.rb * a.nchunk + sb.chunk) * 2 * a.np + p;
    jp[0] = jacc;
    jp[(size_t)a.np] = lacc;
  }
}

}  // namespace porta
