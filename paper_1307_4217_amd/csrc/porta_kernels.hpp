// porta_kernels.hpp -- HIP kernels of the forward path for gfx950: table
// preparation, the plane step of the short-characteristics sweep, the
// ray/frequency reduction of J^K_Q and the stand-alone J accumulation (the
// statistical-equilibrium update is in porta_see.hpp).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "porta_math.hpp"

namespace porta {

constexpr int kMaxMu = 64;
constexpr int kUploadChunk = 480;   // doubles per upload launch (kernel-argument copy)

// ---------------------------------------------------------------------------
// Small host -> device uploads travel inside the kernel arguments, which the
// runtime copies at launch time; the host buffer can be reused at once and
// the copy is ordered on the caller's stream.
// ---------------------------------------------------------------------------
struct UploadChunk {
  double v[kUploadChunk];
  double* dst;
  int n;
};

__global__ void k_upload(const UploadChunk c) {
  for (int t = threadIdx.x; t < c.n; t += blockDim.x) c.dst[t] = c.v[t];
}

// Opt-in validity check of the transfer coefficients: flag[0] = 1 if some eta_I is
// not finite or not > 0, or some propagation-matrix or emission entry is not finite.
// Every writer stores the same value, so the unordered stores agree.
__global__ void k_zero_flag(int* flag) {
  if (threadIdx.x == 0) flag[0] = 0;
}

template <class T>
__global__ void __launch_bounds__(256) k_check_fields(const T* __restrict__ kappa,
                                                      const T* __restrict__ prop,
                                                      const T* __restrict__ emis, size_t N,
                                                      int* flag) {
  for (size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x; p < N;
       p += (size_t)gridDim.x * blockDim.x) {
    bool bad = !(kappa[p] > T(0)) || !isfinite(kappa[p]);
#pragma unroll
    for (int c = 0; c < 6; ++c) bad = bad || !isfinite(prop[c * N + p]) || !isfinite(emis[c * N + p]);
    if (bad) flag[0] = 1;
  }
}

__global__ void k_fill_f64(double* __restrict__ p, size_t n, double v) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// Where the points M (side 0) and P (side 1) of a ray lie when it crosses the layer between
// planes l and l + 1: the path length ds to the plane and the displacement (u, v) in cells,
// reduced to one period and split into the node it is taken from (fu, fv; the node below it, or
// the nearest for the 9-point stencil) and the rest (tx, ty).  It is the same for every
// node of the plane, so it is formed once per call, [ray][layer][side]: in each thread of
// the plane step its two square roots' worth of divisions and floors were a fifth of the
// set-up.
struct RayGeom {
  double ds, tx, ty;
  int fu, fv;
};

// Rays [ray0, ray0 + nray) on nl layers, `stride` of them apart from one ray to the next.
struct GeomArgs {
  const double* z;    // device: heights of the layers' nl + 1 planes
  int ray0, nray, nl, stride;
  int nx, ny;
  double inv_dx, inv_dy;
  double half;        // 0 (bilinear) or 0.5 (9-point)
  RayGeom* geom;
};

// Both sides of one ray and layer: entry e of nray * nl.
__device__ inline void make_geom(const GeomArgs& ga, const double* __restrict__ mu, int nh,
                                 int nchi, int e) {
  const int rb = e / ga.nl, r = ga.ray0 + rb, l = e % ga.nl;
  const double m0 = mu[(r % nh) / nchi], chi = (r % nchi + 0.5) * (2.0 * M_PI / nchi);
  const double st = sqrt(fmax(0.0, 1.0 - m0 * m0));
  const double ds = fabs(ga.z[l + 1] - ga.z[l]) * (1.0 / fabs(m0));
  const double sx = st * cos(chi), sy = st * sin(chi);
#pragma unroll
  for (int side = 0; side < 2; ++side) {
    const double d = side == 0 ? -ds : ds;
    const CellShift u = cell_shift(d * sx * ga.inv_dx, ga.nx, ga.half);
    const CellShift v = cell_shift(d * sy * ga.inv_dy, ga.ny, ga.half);
    const RayGeom g = {ds, u.t, v.t, u.f, v.f};
    ga.geom[((size_t)rb * ga.stride + l) * 2 + side] = g;
  }
}

__global__ void __launch_bounds__(256)
    k_geom(const GeomArgs ga, const double* __restrict__ mu, int nh, int nchi) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e < ga.nray * ga.nl) make_geom(ga, mu, nh, nchi, e);
}

constexpr int kMaxFreq = 4096;   // frequencies of a quadrature, at most

// Ray constants (direction, weight, emission and J projection tables) and the normalized
// frequency weights (block 0), and the rays' geometry (the other blocks), from the uploaded
// quadrature and plane heights.
template <class T>
__global__ void __launch_bounds__(256)
    k_prepare(const double* __restrict__ mu, const double* __restrict__ wmu, int nmu, int nchi,
              double w2, const double* __restrict__ phi, const double* __restrict__ wfreq,
              int nfreq, RayConsts* __restrict__ rays, T* __restrict__ phiT,
              double* __restrict__ wn, const GeomArgs ga) {
  __shared__ double prod[kMaxFreq];
  __shared__ double norm;
  const int nh = nmu * nchi;
  if (blockIdx.x > 0) {
    const int e = (blockIdx.x - 1) * blockDim.x + threadIdx.x;
    if (e < ga.nray * ga.nl) make_geom(ga, mu, nh, nchi, e);
    return;
  }
  for (int r = threadIdx.x; r < 2 * nh; r += blockDim.x) {
    const int a = (r % nh) / nchi, m = r % nchi;
    const double m0 = mu[a];
    const double chi = (m + 0.5) * (2.0 * M_PI / nchi);
    ray_consts(r < nh ? m0 : -m0, chi, 0.5 * wmu[a] / nchi, w2, rays[r]);
  }
  for (int j = threadIdx.x; j < nfreq; j += blockDim.x) prod[j] = wfreq[j] * phi[j];
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int j = 0; j < nfreq; ++j) s += prod[j];
    norm = s;
  }
  __syncthreads();
  for (int j = threadIdx.x; j < nfreq; j += blockDim.x) {
    wn[j] = prod[j] / norm;
    phiT[j] = (T)phi[j];
  }
}

// ---------------------------------------------------------------------------
// Vector loads and stores of one Stokes vector.
// ---------------------------------------------------------------------------
__device__ inline void load4(const float* p, float v[4]) {
  const float4 q = *reinterpret_cast<const float4*>(p);
  v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
}
__device__ inline void load4(const double* p, double v[4]) {
  const double2 a = *reinterpret_cast<const double2*>(p);
  const double2 b = *reinterpret_cast<const double2*>(p + 2);
  v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
}
__device__ inline void store4(float* p, const float v[4]) {
  *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
}
__device__ inline void store4(double* p, const double v[4]) {
  *reinterpret_cast<double2*>(p) = make_double2(v[0], v[1]);
  *reinterpret_cast<double2*>(p + 2) = make_double2(v[2], v[3]);
}
// The same with the non-temporal hint: a plane state that the next launch reads from
// HBM anyway (the planes of a launch exceed the caches) need not take L2 lines from
// the upwind rows and coefficients that neighbouring tiles read again.
typedef float porta_f4 __attribute__((ext_vector_type(4)));
typedef double porta_d2 __attribute__((ext_vector_type(2)));
__device__ inline void store4_nt(float* p, const float v[4]) {
  const porta_f4 q = {v[0], v[1], v[2], v[3]};
  __builtin_nontemporal_store(q, reinterpret_cast<porta_f4*>(p));
}
__device__ inline void store4_nt(double* p, const double v[4]) {
  const porta_d2 a = {v[0], v[1]}, b = {v[2], v[3]};
  __builtin_nontemporal_store(a, reinterpret_cast<porta_d2*>(p));
  __builtin_nontemporal_store(b, reinterpret_cast<porta_d2*>(p + 2));
}

__device__ inline int wrapi(int v, int n) {
  v %= n;
  return v < 0 ? v + n : v;
}

// Bilinear stencil on a periodic plane for a point displaced from node (i, j).  For one ray
// and one pair of planes the displacement is the same at every node, so every thread of a
// plane sees the same weights.
struct Stencil {
  int i00, i10, i01, i11;
  double w00, w10, w01, w11;
};

// Index i + f on a periodic axis of n nodes, for i in [0, n), f in [0, n].
__device__ inline int shift_index(int i, int f, int n) {
  const int v = i + f;
  return v >= n ? v - n : v;
}

__device__ inline Stencil stencil_at(int i0, int i1, int j0, int j1, int nx, double tx,
                                     double ty) {
  Stencil s;
  s.i00 = j0 * nx + i0;
  s.i10 = j0 * nx + i1;
  s.i01 = j1 * nx + i0;
  s.i11 = j1 * nx + i1;
  s.w00 = (1.0 - tx) * (1.0 - ty);
  s.w10 = tx * (1.0 - ty);
  s.w01 = (1.0 - tx) * ty;
  s.w11 = tx * ty;
  return s;
}

__device__ inline Stencil make_stencil(int i, int j, int nx, int ny, const RayGeom& g) {
  const int i0 = shift_index(i, g.fu, nx), j0 = shift_index(j, g.fv, ny);
  return stencil_at(i0, i0 + 1 == nx ? 0 : i0 + 1, j0, j0 + 1 == ny ? 0 : j0 + 1, nx, g.tx, g.ty);
}

// The same for a displacement (u, v) in cells.
__device__ inline Stencil make_stencil(int i, int j, int nx, int ny, double u, double v) {
  const CellShift su = cell_shift(u, nx, 0.0), sv = cell_shift(v, ny, 0.0);
  const RayGeom g = {0.0, su.t, sv.t, su.f, sv.f};
  return make_stencil(i, j, nx, ny, g);
}

template <class T>
__device__ inline double bil(const T* __restrict__ f, const Stencil& s) {
  return fma_t(s.w11, (double)f[s.i11],
               dot3(s.w10, (double)f[s.i10], s.w00, (double)f[s.i00], s.w01, (double)f[s.i01]));
}

// Transposed stencil: the nodes (i', j') whose stencil for the same displacement contains
// node (i, j), with the weight that node received.  Used by the adjoint to turn the
// scatter of the forward interpolation into a gather.
__device__ inline Stencil make_tstencil(int i, int j, int nx, int ny, const RayGeom& g) {
  const int i0 = i - g.fu < 0 ? i - g.fu + nx : i - g.fu;   // f in [0, n]
  const int j0 = j - g.fv < 0 ? j - g.fv + ny : j - g.fv;
  return stencil_at(i0, i0 == 0 ? nx - 1 : i0 - 1, j0, j0 == 0 ? ny - 1 : j0 - 1, nx, g.tx, g.ty);
}

// 3x3 stencil around the node nearest to the displaced point (mode B), with the
// fractional offsets tx, ty in [-1/2, 1/2) from that node.
struct Stencil9 {
  int col[3];     // x indices of columns -1, 0, +1 (periodic)
  int row[3];     // offsets j * nx of rows -1, 0, +1 (periodic)
  double tx, ty;
};

__device__ inline Stencil9 make_stencil9(int i, int j, int nx, int ny, const RayGeom& g) {
  Stencil9 s;
  s.tx = g.tx;
  s.ty = g.ty;
  const int ic = shift_index(i, g.fu, nx), jc = shift_index(j, g.fv, ny);
  s.col[0] = (ic == 0) ? nx - 1 : ic - 1;
  s.col[1] = ic;
  s.col[2] = (ic + 1 == nx) ? 0 : ic + 1;
  s.row[0] = ((jc == 0) ? ny - 1 : jc - 1) * nx;
  s.row[1] = jc * nx;
  s.row[2] = ((jc + 1 == ny) ? 0 : jc + 1) * nx;
  return s;
}

// Monotonic Bezier interpolation on a plane: along x for each of the three rows,
// then along y.
template <class T>
__device__ inline double bez9(const T* __restrict__ f, const Stencil9& s) {
  const BezW<double> wx = bez_weights(s.tx), wy = bez_weights(s.ty);
  double r[3];
#pragma unroll
  for (int b = 0; b < 3; ++b) {
    const T* row = f + s.row[b];
    r[b] = bez_eval(wx, (double)row[s.col[0]], (double)row[s.col[1]], (double)row[s.col[2]]);
  }
  return bez_eval(wy, r[0], r[1], r[2]);
}

// bez9 of a coefficient that is first used behind a branch.  The compiler moves the arithmetic
// behind the branch as well, and nine values loaded stay where one would: of an FP64 sweep 94
// registers, each stored to scratch memory as soon as it was there.  The empty asm takes
// the result at its place.  FP64 sweeps of 9 planes with and without, 16 rays 200x200, 1, 4 and 60
// frequencies 1.59, 3.16; 2.13, 3.73; 12.9, 14.4 ms; FP32, which has the registers, 1.35, 1.32;
// 1.69, 1.66; 7.30, 7.27, so left to the compiler.
template <class T>
__device__ inline double bez9_here(const T* __restrict__ f, const Stencil9& s) {
  double v = bez9(f, s);
  if constexpr (sizeof(T) == 8) asm volatile("" : "+v"(v));
  return v;
}

// Frequency-independent part of the update of node p on plane kO for one ray:
// transfer coefficients interpolated at M (plane kM) and P (plane kP, if any),
// source vectors S = eps/eta_I at M, O, P, K' at M and O, the line-centre
// optical paths and the BESSER control points (Sect. 3.1-3.3).  The multipoles K = 0, 2
// give Stokes V no emission, so the source vectors have three components.
struct PointSetup {
  Stencil sM;
  double dsM, dsP;
  double kapM, kapO, kapP, ikM, ikO, ikP;
  double epsM[6], epsO[6], epsP[6], etaM[6], etaO[6];
  double SM[3], SO[3], SP[3], cM[3];
  double tau0M, tau0P, ratio, lamfac;
  bool hasP;
};

// Emission sum_c emis[s][c] eps_c of I, Q, U; the K = 0 multipole emits in I only and the
// Q = 0 one of K = 2 not in U.
__device__ inline void emission(const RayConsts& rc, const double eps[6], double e[3]) {
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    double v = rc.emis[s][s] * eps[s];
#pragma unroll
    for (int c = s + 1; c < 6; ++c) v = fma_t(rc.emis[s][c], eps[c], v);
    e[s] = v;
  }
}

// The rest of the set-up from the coefficients and path lengths at M, O and P.
// lamfac: Lambda* = omega_O + lamfac omega_C for a unit source at O alone (Eq. 14): c_M is 1
// for BESSER, (1 + ratio)/2 for the parabola, 1/2 without a downwind point.
__device__ inline void setup_sources(const RayConsts& rc, bool parabolic, PointSetup& ps) {
  ps.ikM = 1.0 / ps.kapM;
  ps.ikO = 1.0 / ps.kapO;
  double e[3];
  emission(rc, ps.epsM, e);
#pragma unroll
  for (int s = 0; s < 3; ++s) ps.SM[s] = e[s] * ps.ikM;
  emission(rc, ps.epsO, e);
#pragma unroll
  for (int s = 0; s < 3; ++s) ps.SO[s] = e[s] * ps.ikO;
  ps.tau0M = 0.5 * (ps.kapM + ps.kapO) * ps.dsM;   // line-centre tau_MO
  if (ps.hasP) {
    ps.ikP = 1.0 / ps.kapP;
    emission(rc, ps.epsP, e);
    ps.tau0P = 0.5 * (ps.kapO + ps.kapP) * ps.dsP;
    const double r = ps.tau0M / ps.tau0P, inv = 0.5 / (1.0 + r), ir = 1.0 / r;
    ps.ratio = r;
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      ps.SP[s] = e[s] * ps.ikP;
      ps.cM[s] = control_cm(ps.SM[s], ps.SO[s], ps.SP[s], fma_t(e[s], ps.ikP, -ps.SO[s]), r, inv,
                            ir, parabolic);
    }
    ps.lamfac = parabolic ? control_cm(0.0, 1.0, 0.0, -1.0, r, inv, ir, true) : 1.0;
  } else {
    // no downwind plane: linear control point
    ps.dsP = ps.kapP = ps.ikP = ps.tau0P = ps.ratio = 0.0;
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      ps.SP[s] = 0.0;
      ps.cM[s] = 0.5 * (ps.SM[s] + ps.SO[s]);
    }
#pragma unroll
    for (int c = 0; c < 6; ++c) ps.epsP[c] = 0.0;
    ps.lamfac = 0.5;
  }
}

// gM, gP: the geometry of the layers to kM and kP (gP unused without kP).
template <int MODE, class T>
__device__ inline void setup_point(const T* __restrict__ kappa, const T* __restrict__ prop,
                                   const T* __restrict__ emis, size_t N, int nx, int ny, int np,
                                   int kO, int kM, int kP, const RayGeom& gM, const RayGeom& gP,
                                   const RayConsts& rc, int p, bool parabolic, PointSetup& ps,
                                   Stencil9& sM9) {
  const int j = p / nx, i = p - j * nx;
  const size_t bM = (size_t)kM * np, bO = (size_t)kO * np + p;
  ps.dsM = gM.ds;
  if (MODE == 0) {
    ps.sM = make_stencil(i, j, nx, ny, gM);
    ps.kapM = bil(kappa + bM, ps.sM);
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      ps.epsM[c] = bil(emis + c * N + bM, ps.sM);
      ps.etaM[c] = bil(prop + c * N + bM, ps.sM);
    }
  } else {
    ps.sM = Stencil{0, 0, 0, 0, 1.0, 0.0, 0.0, 0.0};
    sM9 = make_stencil9(i, j, nx, ny, gM);
    ps.kapM = bez9_here(kappa + bM, sM9);
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      ps.epsM[c] = bez9_here(emis + c * N + bM, sM9);
      ps.etaM[c] = bez9_here(prop + c * N + bM, sM9);
    }
  }
  ps.kapO = (double)kappa[bO];
#pragma unroll
  for (int c = 0; c < 6; ++c) {
    ps.epsO[c] = (double)emis[c * N + bO];
    ps.etaO[c] = (double)prop[c * N + bO];
  }
  ps.hasP = kP >= 0;
  if (ps.hasP) {
    ps.dsP = gP.ds;
    const size_t bP = (size_t)kP * np;
    if (MODE == 0) {
      const Stencil sP = make_stencil(i, j, nx, ny, gP);
      ps.kapP = bil(kappa + bP, sP);
#pragma unroll
      for (int c = 0; c < 6; ++c) ps.epsP[c] = bil(emis + c * N + bP, sP);
    } else {
      const Stencil9 sP = make_stencil9(i, j, nx, ny, gP);
      ps.kapP = bez9(kappa + bP, sP);
#pragma unroll
      for (int c = 0; c < 6; ++c) ps.epsP[c] = bez9(emis + c * N + bP, sP);
    }
  }
  setup_sources(rc, parabolic, ps);
}

// Geometry of the layer between planes k and k2 for one ray and side (0: M, 1: P), from a
// table of nz - 1 layers a ray.
__device__ inline const RayGeom& layer_geom(const RayGeom* __restrict__ geom, int ray, int nz,
                                            int k, int k2, int side) {
  return geom[((size_t)ray * (nz - 1) + (k < k2 ? k : k2)) * 2 + side];
}

// ---------------------------------------------------------------------------
// One hemisphere's part of a plane step: the plane its rays are solved on, their states,
// and the previous plane's partial sums of J.
// ---------------------------------------------------------------------------
template <class T>
struct HemiArgs {
  const T* iprev;    // upwind plane state, or nullptr when the upwind plane is the boundary
  T* inext;          // state of plane kO
  double* jpart;     // [ray][chunk][NS + 1][node]: sum_j W_j I_i and sum_j W_j Lambda* over
                     // the chunk's frequencies, or nullptr
  const double* jpart_prev;  // partial sums of the previous plane, or nullptr (boundary plane)
  size_t prev_off;   // offset of the previous plane in jkq
  int kO, kM, kP;    // plane of O, upwind plane, downwind plane (-1: none)
  int ray0, nrb;     // rays [ray0, ray0 + nrb) of the enumeration
  T ibound;          // Stokes I on the boundary plane of this hemisphere
};

// ---------------------------------------------------------------------------
// Add the frequency-integrated Stokes vectors of a batch of rays on one plane to J^K_Q
// (Eq. 1) and Lbar, in a fixed order (no atomics).  A block takes kJNodes nodes.  With one
// thread per node and a load per ray in turn the chain of memory latencies took 25 us at 16x16
// nodes and 40 rays, 73 us at 128x128 and 80 rays: more than the plane step that had to wait
// for it.  Two splits, by the precision of the sweep:
// - FP64: groups of rays, added at the end (jreduce_groups).
// - FP32: the rays one by one in the order of the enumeration (jreduce_ordered).  There the
//   next iteration's emissivities are rounded to FP32, and a sum whose last bit differs moves
//   some of them by 6e-8.  The threads, as (ray of a slab, node), load the slab's partial sums
//   and the rays' coefficients into LDS, and then, as (component, node), add its rays in
//   order, while the next slab's loads are under way.
//   Planes that have launches for it: a node a thread (jreduce_serial).
// (FP64 in the second split: 16x16x32 and 80 rays, 537 us a sweep instead of 459; 64x64x49
// multigrid cycles 54.6 ms instead of 54.0.)
// On the boundary plane the Stokes vector is (ibound, 0, 0, 0) at every frequency.  NS: Stokes
// parameters in the partial sums (4, or 1: intensity only).
// ---------------------------------------------------------------------------
constexpr int kJNodes = 16;   // consecutive nodes of a block: one 128-byte line of doubles
constexpr int kJCoefs = 37;   // of a ray: weight and proj[9][4]
inline int jblocks(int np, int nodes = kJNodes) { return (np - 1) / nodes + 1; }
// LDS for `threads` threads: a slab of threads / kJNodes rays, or ten sums of every thread
inline size_t jlds_bytes(int threads, size_t elem) {
  return (size_t)(threads / kJNodes) * (elem == 4 ? 5 * kJNodes + kJCoefs : 10 * kJNodes) *
         sizeof(double);
}

// The partial sums of one plane.
struct JJob {
  const double* part;     // [ray][chunk][NS + 1][node], or nullptr: the boundary plane
  const RayConsts* rays;  // of the batch
  int nrb, nchunk;
  double ibound;
  size_t off;             // of the plane in jkq
};

// In the order of the rays, each of one chunk.
template <int NS>
__device__ inline void jreduce_ordered(const JJob& J, double* __restrict__ jkq, size_t N, int np,
                                       int node0, double* lds, int threads) {
  constexpr int NV = NS + 1;
  const int G = threads / kJNodes;
  const int g = threadIdx.x / kJNodes, n = threadIdx.x % kJNodes, p = node0 + n;
  const bool works = (int)threadIdx.x < threads;
  double* s_part = lds;                            // [ray][NV][node]
  double* s_coef = lds + (size_t)G * 5 * kJNodes;  // [ray][kJCoefs]
  constexpr int kTasks = 10 * kJNodes, kMaxTasks = (kTasks + 63) / 64;   // of a thread
  constexpr int kMaxCoefs = (kJCoefs + kJNodes - 1) / kJNodes;
  double acc[kMaxTasks];
#pragma unroll
  for (int k = 0; k < kMaxTasks; ++k) acc[k] = 0.0;
  double v[NV], cf[kMaxCoefs];
  // Rays past the batch's last are zeros, which the unrolled loop below adds.
  auto load = [&](int r0) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < kMaxCoefs; ++k) {
      const int e = threadIdx.x + k * threads, r = e / kJCoefs, q = e - r * kJCoefs;
      cf[k] = 0.0;
      if (r < G && r0 + r < J.nrb) {
        const RayConsts& rc = J.rays[r0 + r];
        cf[k] = *(q == 0 ? &rc.weight : &rc.proj[0][0] + (q - 1));
      }
    }
    const int rb = r0 + g;
#pragma unroll
    for (int s = 0; s < NV; ++s) v[s] = 0.0;
    if (rb >= J.nrb || p >= np) return;
    if (!J.part) {
      v[0] = J.ibound;
      return;
    }
    const double* jp = J.part + (size_t)rb * NV * np + p;   // one chunk
#pragma unroll
    for (int s = 0; s < NV; ++s) v[s] = jp[s * (size_t)np];
  };
  if (works) load(0);
  for (int r0 = 0; r0 < J.nrb; r0 += G) {
    const int nr = min(G, J.nrb - r0);
    if (works) {
#pragma unroll
      for (int s = 0; s < NV; ++s) s_part[(g * NV + s) * kJNodes + n] = v[s];
#pragma unroll
      for (int k = 0; k < kMaxCoefs; ++k) {
        const int e = threadIdx.x + k * threads;
        if (e < G * kJCoefs) s_coef[e] = cf[k];
      }
    }
    __syncthreads();
    if (works) load(r0 + G);
    if (works) {
#pragma unroll
      for (int k = 0; k < kMaxTasks; ++k) {
        const int e = threadIdx.x + k * threads;
        if (e < kTasks) {
          const int c = e / kJNodes;
          const double* part = s_part + e % kJNodes;
          const double* coef = s_coef + (c < 9 ? 1 + 4 * c : 0);
          const double* weight = s_coef;
          for (int r = 0; r < nr; r += 4) {   // G is a multiple of 4
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              double x;
              if constexpr (NS == 4) {
                x = dot3(coef[1], part[kJNodes], coef[0], part[0], coef[2], part[2 * kJNodes]);
                x = fma_t(coef[3], part[3 * kJNodes], x);
              } else {
                x = coef[0] * part[0];
              }
              acc[k] = fma_t(*weight, c == 9 ? part[NS * kJNodes] : x, acc[k]);
              part += NV * kJNodes;
              coef += kJCoefs;
              weight += kJCoefs;
            }
          }
        }
      }
    }
    __syncthreads();
  }
  if (!works) return;
#pragma unroll
  for (int k = 0; k < kMaxTasks; ++k) {
    const int e = threadIdx.x + k * threads, q = node0 + e % kJNodes;
    if (e < kTasks && q < np) jkq[(e / kJNodes) * N + J.off + q] += acc[k];
  }
}

// Group g of the threads, (group, node), adds rays g, g + G, ..., and the groups are added
// through LDS: no barrier between the loads of one ray and the next's, and the projections on
// all the threads.  W: nodes of the block.
template <int NS, int W>
__device__ inline void jreduce_groups(const JJob& J, double* __restrict__ jkq, size_t N, int np,
                                      int node0, double* lds, int threads) {
  constexpr int NV = NS + 1;
  const int G = threads / W;
  // (a group of whole wavefronts: the same ray for all lanes, its constants by scalar loads)
  const int g = W < 64 ? (int)threadIdx.x / W
                       : __builtin_amdgcn_readfirstlane((int)threadIdx.x / W);
  const int n = threadIdx.x % W, p = node0 + n;
  const bool works = (int)threadIdx.x < threads;
  double acc[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  if (works && p < np) {
#pragma unroll W < 64 ? 1 : 2
    for (int rb = g; rb < J.nrb; rb += G) {
      double v[NV];
#pragma unroll
      for (int s = 0; s < NV; ++s) v[s] = 0.0;
      if (!J.part) {
        v[0] = J.ibound;
      } else {
        const double* jp = J.part + (size_t)rb * J.nchunk * NV * np + p;
#pragma unroll 4
        for (int c = 0; c < J.nchunk; ++c) {
#pragma unroll
          for (int s = 0; s < NV; ++s) v[s] += jp[s * (size_t)np];
          jp += NV * (size_t)np;
        }
      }
      const RayConsts& rc = J.rays[rb];
      const double w = rc.weight;
#pragma unroll
      for (int c = 0; c < 9; ++c) {
        double x = rc.proj[c][0] * v[0];
        if constexpr (NS == 4)
          x = fma_t(rc.proj[c][3], v[3], fma_t(rc.proj[c][2], v[2], fma_t(rc.proj[c][1], v[1], x)));
        acc[c] = fma_t(w, x, acc[c]);
      }
      acc[9] = fma_t(w, v[NS], acc[9]);
    }
  }
  if (works) {
#pragma unroll
    for (int c = 0; c < 10; ++c) lds[(c * G + g) * W + n] = acc[c];
  }
  __syncthreads();
  if (!works) return;
  for (int e = threadIdx.x; e < 10 * W; e += threads) {
    const int c = e / W, q = node0 + e % W;
    double sum = 0.0;
    for (int k = 0; k < G; ++k) sum += lds[(c * G + k) * W + e % W];
    if (q < np) jkq[c * N + J.off + q] += sum;
  }
}

// Thread per node: few rays in order, on planes whose nodes fill the chip.  The sums of
// jreduce_ordered, operation by operation.
template <int NS>
__device__ inline void jreduce_serial(const JJob& J, double* __restrict__ jkq, size_t N, int np,
                                      int p) {
  constexpr int NV = NS + 1;
  if (p >= np) return;
  double acc[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll 4
  for (int rb = 0; rb < J.nrb; ++rb) {
    double v[NV];
#pragma unroll
    for (int s = 0; s < NV; ++s) v[s] = 0.0;
    if (!J.part) {
      v[0] = J.ibound;
    } else {
      const double* jp = J.part + (size_t)rb * NV * np + p;   // one chunk
#pragma unroll
      for (int s = 0; s < NV; ++s) v[s] = jp[s * (size_t)np];
    }
    const RayConsts& rc = J.rays[rb];
    const double w = rc.weight;
#pragma unroll
    for (int c = 0; c < 9; ++c) {
      double x;
      if constexpr (NS == 4) {
        x = dot3(rc.proj[c][1], v[1], rc.proj[c][0], v[0], rc.proj[c][2], v[2]);
        x = fma_t(rc.proj[c][3], v[3], x);
      } else {
        x = rc.proj[c][0] * v[0];
      }
      acc[c] = fma_t(w, x, acc[c]);
    }
    acc[9] = fma_t(w, v[NS], acc[9]);
  }
#pragma unroll
  for (int c = 0; c < 10; ++c) jkq[c * N + J.off + p] += acc[c];
}

// Every thread of the block calls it; the first `threads` of them work.  T: precision of the
// sweep; W: nodes of the block (FP32: kJNodes, or a node a thread).
template <int NS, class T, int W = kJNodes>
__device__ inline void jreduce_block(const JJob& J, double* __restrict__ jkq, size_t N, int np,
                                     int node0, double* lds, int threads) {
  if constexpr (sizeof(T) == 4 && W == kJNodes)
    jreduce_ordered<NS>(J, jkq, N, np, node0, lds, threads);
  else if constexpr (sizeof(T) == 4)
    jreduce_serial<NS>(J, jkq, N, np, node0 + (int)threadIdx.x);
  else
    jreduce_groups<NS, W>(J, jkq, N, np, node0, lds, threads);
}

// first: the first block's place among the plane's blocks of W nodes.
template <int NS, class T, int W>
__global__ void __launch_bounds__(256)
    k_jreduce(const JJob J, double* __restrict__ jkq, int np, size_t N, int first) {
  extern __shared__ double s_tab[];
  jreduce_block<NS, T, W>(J, jkq, N, np, (first + (int)blockIdx.x) * W, s_tab, blockDim.x);
}

// ---------------------------------------------------------------------------
// One plane step of the sweep for a batch of rays and every frequency: the upward rays
// (h[0]) on their plane and the downward rays (h[1]) on theirs, which are independent
// of each other.  Thread = (node, ray, chunk of frequencies); the frequency loop runs
// inside the thread so that the frequency-independent work (interpolation of the
// coefficients at M and P, S and K' at M and O, the BESSER control points) is done
// once per node, ray and chunk.  One chunk holds every frequency unless the launch
// would leave most of the chip idle (sweep_plan on the host).
//
// The last njb blocks add the previous plane's partial sums to J: where the launch takes
// several rounds of the chip they fill its tail, and otherwise they run beside the others.
//
// Plane state layout: [ray in batch][frequency][node][Stokes].
// ---------------------------------------------------------------------------
template <class T>
struct PlaneArgs {
  const T* kappa;
  const T* prop;
  const T* emis;
  const RayConsts* rays;
  const RayGeom* geom;
  const T* phi;
  const double* wn;
  HemiArgs<T> h[2];
  double* jkq;       // [10][N] or nullptr
  size_t N;
  int nx, ny;
  int nz;            // of the geometry table (layer_geom)
  int np, nfreq;
  int ntile;         // tiles of blockDim.x nodes in a plane
  int nchunk, fchunk;
  int nstep;         // blocks of the plane step; the J reduction's follow
  int njb;           // blocks of the J reduction
  int jsame;         // both hemispheres' previous plane is the same one: one block adds both
  int xcd_remap;     // tiles per XCD per round (0: hardware order), see xcd_order
  int parabolic;     // control point: 0 BESSER, 1 parabola through M, O, P
};

// The arguments of one hemisphere, field by field: an index into an array of them taken at run
// time would leave the pointers without their address space (flat loads and stores, 2% of
// the sweep at 256x256x128).
template <class T>
__device__ inline HemiArgs<T> hemi_pick(const HemiArgs<T>& u, const HemiArgs<T>& d, bool second) {
  HemiArgs<T> h;
  h.iprev = second ? d.iprev : u.iprev;
  h.inext = second ? d.inext : u.inext;
  h.jpart = second ? d.jpart : u.jpart;
  h.jpart_prev = second ? d.jpart_prev : u.jpart_prev;
  h.prev_off = second ? d.prev_off : u.prev_off;
  h.kO = second ? d.kO : u.kO;
  h.kM = second ? d.kM : u.kM;
  h.kP = second ? d.kP : u.kP;
  h.ray0 = second ? d.ray0 : u.ray0;
  h.nrb = second ? d.nrb : u.nrb;
  h.ibound = second ? d.ibound : u.ibound;
  return h;
}
template <class T>
__device__ inline HemiArgs<T> hemi_args(const PlaneArgs<T>& a, bool second) {
  return hemi_pick(a.h[0], a.h[1], second);
}

// The J reduction of the previous planes by the last njb blocks of a plane step: half of
// them for each hemisphere.
template <int NS, class T>
__device__ inline void jblock(const PlaneArgs<T>& a, double* lds) {
  const int b = blockIdx.x - a.nstep, per = a.njb / 2, hemi = b >= per;
  const int node0 = (b - hemi * per) * kJNodes;
  const HemiArgs<T> h = hemi_args(a, hemi);
  if (node0 >= a.np || h.nrb == 0 || (hemi && a.jsame)) return;
  const JJob j = {h.jpart_prev, a.rays + h.ray0, h.nrb, a.nchunk, (double)h.ibound, h.prev_off};
  jreduce_block<NS, T>(j, a.jkq, a.N, a.np, node0, lds, blockDim.x);
  if (a.jsame) {
    __syncthreads();   // the first one's LDS has been read
    const HemiArgs<T>& d = a.h[1];
    const JJob k = {d.jpart_prev, a.rays + d.ray0, d.nrb, a.nchunk, (double)d.ibound, h.prev_off};
    jreduce_block<NS, T>(k, a.jkq, a.N, a.np, node0, lds, blockDim.x);
  }
}

// Workgroups are dispatched round-robin over the 8 XCDs of the MI355X, each with
// its own L2.  With chunk R > 0 the tiles are renumbered so that every XCD takes
// R consecutive tiles per round (neighbouring rows of one ray then share an L2)
// while the eight XCDs still advance through the grid together.
__device__ inline int xcd_order(int chunk, int L, int T) {
  int Lp = L;
  if (chunk > 0) {
    const int round = 8 * chunk;
    const int Tmain = (T / round) * round;
    if (L < Tmain) {
      const int x = L % 8, k = L / 8;
      Lp = (k / chunk) * round + x * chunk + (k % chunk);
    }
  }
  return Lp;
}

// Tile, ray, frequency chunk and hemisphere of a block of a plane step.
struct StepBlock {
  int bx, rb, chunk, hemi;   // rb counts within the hemisphere's rays
};

template <class T>
__device__ inline StepBlock step_block(const PlaneArgs<T>& a) {
  const int L = xcd_order(a.xcd_remap, blockIdx.x, a.nstep);
  const int row = L / a.ntile, ray = row / a.nchunk;
  StepBlock b;
  b.bx = L % a.ntile;
  b.chunk = row % a.nchunk;
  b.hemi = ray >= a.h[0].nrb;
  b.rb = ray - (b.hemi ? a.h[0].nrb : 0);
  return b;
}

template <class T>
__device__ inline void load_upwind(const T* __restrict__ q, const Stencil& s, T v[4][4]) {
  load4(q + 4 * (size_t)s.i00, v[0]);
  load4(q + 4 * (size_t)s.i10, v[1]);
  load4(q + 4 * (size_t)s.i01, v[2]);
  load4(q + 4 * (size_t)s.i11, v[3]);
}

// Upwind Stokes vector of one frequency by the 9-point monotonic Bezier (mode B).
template <class T>
__device__ inline void upwind_bez9(const T* __restrict__ q, const Stencil9& s,
                                   const BezW<T>& wx, const BezW<T>& wy, T IM[4]) {
  T v[3][3][4];
#pragma unroll
  for (int b = 0; b < 3; ++b)
#pragma unroll
    for (int a = 0; a < 3; ++a) load4(q + 4 * (size_t)(s.row[b] + s.col[a]), v[b][a]);
#pragma unroll
  for (int st = 0; st < 4; ++st) {
    T r[3];
#pragma unroll
    for (int b = 0; b < 3; ++b) r[b] = bez_eval(wx, v[b][0][st], v[b][1][st], v[b][2][st]);
    IM[st] = bez_eval(wy, r[0], r[1], r[2]);
  }
}

template <class T>
__device__ inline T bilinear(T w00, T w10, T w01, T w11, T v00, T v10, T v01, T v11) {
  return fma_t(w11, v11, dot3(w00, v00, w10, v10, w01, v01));
}

// Entries (e, r) of K' = K / eta_I - 1 in the sweep precision.
template <class T>
__device__ inline void kprime_entries(const double eta[6], double ik, T e[3], T r[3]) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    e[c] = (T)(eta[c] * ik);
    r[c] = (T)(eta[3 + c] * ik);
  }
}

// The right-hand side of Eq. fsbez with Eq. kappa, (e - psi'_M K'_M) I_M + sources, with
// KI = K'_M I_M; Stokes V has no source.
template <class T>
__device__ inline void step_rhs(const Coefs<T>& cf, const T IM[4], const T KI[4],
                                const StepSource<T> src[3], T b[4]) {
  const StepSource<T> w = source_weights(cf);
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    b[s] = fma_t(cf.e, IM[s], -(cf.psiM * KI[s]));
    if (s < 3) b[s] = add_sources(w, src[s], b[s]);
  }
}

// Occupancy targets: three waves per SIMD for the FP32 bilinear sweep (168 VGPRs,
// with the next frequency's corners in flight and no spill in the loop; four or five
// waves were slower), two for the others (the 9-point mode would otherwise drop to
// one).
template <class T, int MODE>
__global__ void __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(MODE == 0 && sizeof(T) == 4 ? 3 : 2,
                                   MODE == 0 && sizeof(T) == 4 ? 3 : 2)))
k_sweep_plane(const PlaneArgs<T> a) {
  // per-frequency weights and profile, read from LDS inside the frequency loop so that
  // no vector-memory wait (which on gfx9 also covers earlier stores) sits in the loop
  extern __shared__ double s_tab[];
  if ((int)blockIdx.x >= a.nstep) {
    jblock<4>(a, s_tab);
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
  const RayConsts& rc = a.rays[h.ray0 + sb.rb];
  PointSetup ps;
  Stencil9 sM9;
  const int ray = h.ray0 + sb.rb;
  setup_point<MODE>(a.kappa, a.prop, a.emis, a.N, a.nx, a.ny, a.np, h.kO, h.kM, h.kP,
                    layer_geom(a.geom, ray, a.nz, h.kO, h.kM, 0),
                    layer_geom(a.geom, ray, a.nz, h.kO, h.kP < 0 ? h.kM : h.kP, 1), rc, p,
                    a.parabolic != 0, ps, sM9);
  const BezW<T> bwx = bez_weights(MODE == 1 ? (T)sM9.tx : T(0));
  const BezW<T> bwy = bez_weights(MODE == 1 ? (T)sM9.ty : T(0));
  const Stencil& sM = ps.sM;

  // frequency-independent pieces in the sweep precision
  T eMv[3], rMv[3], eOv[3], rOv[3];
  kprime_entries(ps.etaM, ps.ikM, eMv, rMv);
  kprime_entries(ps.etaO, ps.ikO, eOv, rOv);
  const auto KO = step_op(eOv, rOv);
  StepSource<T> src[3];
#pragma unroll
  for (int s = 0; s < 3; ++s) step_source(ps.SM[s], ps.SO[s], ps.cM[s], src[s]);
  const T tau0 = (T)ps.tau0M;
  const T w00 = (T)sM.w00, w10 = (T)sM.w10, w01 = (T)sM.w01, w11 = (T)sM.w11;
  const T lf = (T)ps.lamfac;

  const size_t fstride = (size_t)a.np * 4;
  const size_t foff = ((size_t)sb.rb * a.nfreq + f0) * fstride;
  const T* ip = h.iprev ? h.iprev + foff : nullptr;
  T* op = h.inext + foff + (size_t)p * 4;
  double jacc0 = 0.0, jacc1 = 0.0, jacc2 = 0.0, jacc3 = 0.0, lacc = 0.0;

  // one update (Eq. fsbez solved with Eq. kappa) at frequency f0 + f from the upwind
  // Stokes vector IM; odd: of an interior plane's bilinear loop, f is (stokes_solve)
  auto update = [&](int f, T i0, T i1, T i2, T i3, bool odd) __attribute__((always_inline)) {
    const T IM[4] = {i0, i1, i2, i3};
    const Coefs<T> cf = coefficients(tau0 * s_phi[f]);
    T KI[4], b[4], x[4];
    kprime_apply(eMv, rMv, IM, KI);
    step_rhs(cf, IM, KI, src, b);
    stokes_solve<1>(KO, step_freq(KO, cf.psiO), b, x, odd);
    store4_nt(op + (size_t)f * fstride, x);
    const double W = s_wn[f];
    jacc0 = fma_t(W, (double)x[0], jacc0);
    jacc1 = fma_t(W, (double)x[1], jacc1);
    jacc2 = fma_t(W, (double)x[2], jacc2);
    jacc3 = fma_t(W, (double)x[3], jacc3);
    lacc = fma_t(W, (double)lambda_star(cf, lf), lacc);
  };
  // bilinear upwind component s from the four corner values
#define PORTA_BILIN(v, s) bilinear(w00, w10, w01, w11, v[0][s], v[1][s], v[2][s], v[3][s])

  if (!ip) {
    // the upwind plane is the boundary
    for (int f = 0; f < nf; ++f) update(f, h.ibound, T(0), T(0), T(0), false);
  } else if (MODE == 1) {
    for (int f = 0; f < nf; ++f) {
      T IM[4];
      upwind_bez9(ip + (size_t)f * fstride, sM9, bwx, bwy, IM);
      update(f, IM[0], IM[1], IM[2], IM[3], false);
    }
  } else {
    if constexpr (sizeof(T) == 4) {
      // The corners of frequency f + 1 are loaded during the arithmetic of frequency f (in
      // FP64 the second buffer does not fit without spilling).  The loads are never
      // skipped (past the end the last frequency's are taken again): behind a branch the
      // wait for the current corners would have to wait for the new ones too.
      T vA[4][4], vB[4][4];
      load_upwind(ip, sM, vA);
      int f = 0;
      for (; f + 1 < nf; f += 2) {
        load_upwind(ip + (size_t)(f + 1) * fstride, sM, vB);
        update(f, PORTA_BILIN(vA, 0), PORTA_BILIN(vA, 1), PORTA_BILIN(vA, 2),
               PORTA_BILIN(vA, 3), false);
        load_upwind(ip + (size_t)min(f + 2, nf - 1) * fstride, sM, vA);
        update(f + 1, PORTA_BILIN(vB, 0), PORTA_BILIN(vB, 1), PORTA_BILIN(vB, 2),
               PORTA_BILIN(vB, 3), true);
      }
      if (f < nf)
        update(f, PORTA_BILIN(vA, 0), PORTA_BILIN(vA, 1), PORTA_BILIN(vA, 2),
               PORTA_BILIN(vA, 3), false);
    } else {
      T v[4][4];
      for (int f = 0; f < nf; ++f) {
        load_upwind(ip + (size_t)f * fstride, sM, v);
        update(f, PORTA_BILIN(v, 0), PORTA_BILIN(v, 1), PORTA_BILIN(v, 2), PORTA_BILIN(v, 3), false);
      }
    }
  }
#undef PORTA_BILIN
  if (h.jpart) {
    double* jp = h.jpart + ((size_t)sb.rb * a.nchunk + sb.chunk) * 5 * a.np + p;
    jp[0] = jacc0;
    jp[(size_t)a.np] = jacc1;
    jp[2 * (size_t)a.np] = jacc2;
    jp[3 * (size_t)a.np] = jacc3;
    jp[4 * (size_t)a.np] = lacc;
  }
}

// Eq. 1 from a stored block of Stokes vectors [nray][nf][N][4].
template <class T>
__global__ void __launch_bounds__(256)
    k_jkq_accumulate(double* __restrict__ jkq, const T* __restrict__ stokes,
                     const T* __restrict__ lam, const RayConsts* __restrict__ rays,
                     const double* __restrict__ wn, int ray0, int nray, int f0, int nf, size_t N) {
  const size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= N) return;
  double acc[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  for (int r = 0; r < nray; ++r) {
    double ib[4] = {0, 0, 0, 0}, lb = 0.0;
    for (int q = 0; q < nf; ++q) {
      const double W = wn[f0 + q];
      const size_t off = ((size_t)r * nf + q) * N + p;
      T v[4];
      load4(stokes + 4 * off, v);
#pragma unroll
      for (int s = 0; s < 4; ++s) ib[s] += W * (double)v[s];
      if (lam) lb += W * (double)lam[off];
    }
    const RayConsts& rc = rays[ray0 + r];
    const double w = rc.weight;
#pragma unroll
    for (int c = 0; c < 9; ++c)
      acc[c] += w * (rc.proj[c][0] * ib[0] + rc.proj[c][1] * ib[1] + rc.proj[c][2] * ib[2] +
                     rc.proj[c][3] * ib[3]);
    acc[9] += w * lb;
  }
#pragma unroll
  for (int c = 0; c < 10; ++c) jkq[c * N + p] += acc[c];
}

}  // namespace porta
