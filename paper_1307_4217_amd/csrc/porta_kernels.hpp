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
constexpr int kUploadChunk = 240;   // doubles per upload launch (kernel-argument copy)

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
  const int t = threadIdx.x;
  if (t < c.n) c.dst[t] = c.v[t];
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

// Ray constants (direction, weight, emission and J projection tables) and the
// normalized frequency weights, from the uploaded quadrature.
template <class T>
__global__ void k_prepare(const double* __restrict__ mu, const double* __restrict__ wmu, int nmu,
                          int nchi, double w2, const double* __restrict__ phi,
                          const double* __restrict__ wfreq, int nfreq,
                          RayConsts* __restrict__ rays, T* __restrict__ phiT,
                          double* __restrict__ wn) {
  __shared__ double norm;
  const int nh = nmu * nchi;
  for (int r = threadIdx.x; r < 2 * nh; r += blockDim.x) {
    const int a = (r % nh) / nchi, m = r % nchi;
    const double m0 = mu[a];
    const double chi = (m + 0.5) * (2.0 * M_PI / nchi);
    ray_consts(r < nh ? m0 : -m0, chi, 0.5 * wmu[a] / nchi, w2, rays[r]);
  }
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int j = 0; j < nfreq; ++j) s += wfreq[j] * phi[j];
    norm = s;
  }
  __syncthreads();
  for (int j = threadIdx.x; j < nfreq; j += blockDim.x) {
    wn[j] = wfreq[j] * phi[j] / norm;
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

// Bilinear stencil on a periodic plane for a point displaced by (u, v) cells
// from node (i, j).  For one ray and one pair of planes the displacement is
// the same at every node, so every thread of a plane sees the same weights.
struct Stencil {
  int i00, i10, i01, i11;
  double w00, w10, w01, w11;
};

__device__ inline Stencil make_stencil(int i, int j, int nx, int ny, double u, double v) {
  // reduce the displacement to one period first so the integer shift stays in range
  u -= nx * floor(u / nx);
  v -= ny * floor(v / ny);
  const double fu = floor(u), fv = floor(v);
  const double tx = u - fu, ty = v - fv;
  const int i0 = wrapi(i + (int)fu, nx), i1 = (i0 + 1 == nx) ? 0 : i0 + 1;
  const int j0 = wrapi(j + (int)fv, ny), j1 = (j0 + 1 == ny) ? 0 : j0 + 1;
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

template <class T>
__device__ inline double bil(const T* __restrict__ f, const Stencil& s) {
  return s.w00 * (double)f[s.i00] + s.w10 * (double)f[s.i10] + s.w01 * (double)f[s.i01] +
         s.w11 * (double)f[s.i11];
}

// Transposed stencil: the nodes (i', j') whose stencil for the same displacement
// (u, v) contains node (i, j), with the weight that node received.  Used by the
// adjoint to turn the scatter of the forward interpolation into a gather.
__device__ inline Stencil make_tstencil(int i, int j, int nx, int ny, double u, double v) {
  u -= nx * floor(u / nx);
  v -= ny * floor(v / ny);
  const double fu = floor(u), fv = floor(v);
  const double tx = u - fu, ty = v - fv;
  const int i0 = wrapi(i - (int)fu, nx), i1 = (i0 == 0) ? nx - 1 : i0 - 1;
  const int j0 = wrapi(j - (int)fv, ny), j1 = (j0 == 0) ? ny - 1 : j0 - 1;
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

// 3x3 stencil around the node nearest to the displaced point (mode B), with the
// fractional offsets tx, ty in [-1/2, 1/2) from that node.
struct Stencil9 {
  int col[3];     // x indices of columns -1, 0, +1 (periodic)
  int row[3];     // offsets j * nx of rows -1, 0, +1 (periodic)
  double tx, ty;
};

__device__ inline Stencil9 make_stencil9(int i, int j, int nx, int ny, double u, double v) {
  u -= nx * floor(u / nx);
  v -= ny * floor(v / ny);
  const double fu = floor(u + 0.5), fv = floor(v + 0.5);
  Stencil9 s;
  s.tx = u - fu;
  s.ty = v - fv;
  const int ic = wrapi(i + (int)fu, nx), jc = wrapi(j + (int)fv, ny);
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

// Frequency-independent part of the update of node p on plane kO for one ray:
// transfer coefficients interpolated at M (plane kM) and P (plane kP, if any),
// source vectors S = eps/eta_I at M, O, P, K' at M and O, the line-centre
// optical paths and the BESSER control points (Sect. 3.1-3.3).
struct PointSetup {
  Stencil sM;
  double dsM, dsP;
  double kapM, kapO, kapP, ikM, ikO, ikP;
  double epsM[6], epsO[6], epsP[6], etaM[6], etaO[6];
  double SM[4], SO[4], SP[4], cM[4];
  double tau0M, tau0P, ratio;
  bool hasP;
};

template <int MODE, class T>
__device__ inline void setup_point(const T* __restrict__ kappa, const T* __restrict__ prop,
                                   const T* __restrict__ emis, size_t N, int nx, int ny, int np,
                                   int kO, int kM, int kP, double dzM, double dzP, double inv_dx,
                                   double inv_dy, const RayConsts& rc, int p, bool parabolic,
                                   PointSetup& ps, Stencil9& sM9) {
  const int i = p % nx, j = p / nx;
  const double inv_mu = 1.0 / fabs(rc.mu);
  ps.dsM = dzM * inv_mu;
  const double uM = -ps.dsM * rc.sx * inv_dx, vM = -ps.dsM * rc.sy * inv_dy;
  const size_t bM = (size_t)kM * np, bO = (size_t)kO * np + p;
  if (MODE == 0) {
    ps.sM = make_stencil(i, j, nx, ny, uM, vM);
    ps.kapM = bil(kappa + bM, ps.sM);
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      ps.epsM[c] = bil(emis + c * N + bM, ps.sM);
      ps.etaM[c] = bil(prop + c * N + bM, ps.sM);
    }
  } else {
    ps.sM = Stencil{0, 0, 0, 0, 1.0, 0.0, 0.0, 0.0};
    sM9 = make_stencil9(i, j, nx, ny, uM, vM);
    ps.kapM = bez9(kappa + bM, sM9);
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      ps.epsM[c] = bez9(emis + c * N + bM, sM9);
      ps.etaM[c] = bez9(prop + c * N + bM, sM9);
    }
  }
  ps.kapO = (double)kappa[bO];
  ps.ikM = 1.0 / ps.kapM;
  ps.ikO = 1.0 / ps.kapO;
#pragma unroll
  for (int c = 0; c < 6; ++c) {
    ps.epsO[c] = (double)emis[c * N + bO];
    ps.etaO[c] = (double)prop[c * N + bO];
  }
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    double em = 0.0, eo = 0.0;
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      em += rc.emis[s][c] * ps.epsM[c];
      eo += rc.emis[s][c] * ps.epsO[c];
    }
    ps.SM[s] = em * ps.ikM;
    ps.SO[s] = eo * ps.ikO;
  }
  ps.tau0M = 0.5 * (ps.kapM + ps.kapO) * ps.dsM;   // line-centre tau_MO
  ps.hasP = kP >= 0;
  if (ps.hasP) {
    ps.dsP = dzP * inv_mu;
    const double uP = ps.dsP * rc.sx * inv_dx, vP = ps.dsP * rc.sy * inv_dy;
    const size_t bP = (size_t)kP * np;
    if (MODE == 0) {
      const Stencil sP = make_stencil(i, j, nx, ny, uP, vP);
      ps.kapP = bil(kappa + bP, sP);
#pragma unroll
      for (int c = 0; c < 6; ++c) ps.epsP[c] = bil(emis + c * N + bP, sP);
    } else {
      const Stencil9 sP = make_stencil9(i, j, nx, ny, uP, vP);
      ps.kapP = bez9(kappa + bP, sP);
#pragma unroll
      for (int c = 0; c < 6; ++c) ps.epsP[c] = bez9(emis + c * N + bP, sP);
    }
    ps.ikP = 1.0 / ps.kapP;
    ps.tau0P = 0.5 * (ps.kapO + ps.kapP) * ps.dsP;
    ps.ratio = ps.tau0M / ps.tau0P;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      double ep = 0.0;
#pragma unroll
      for (int c = 0; c < 6; ++c) ep += rc.emis[s][c] * ps.epsP[c];
      ps.SP[s] = ep * ps.ikP;
      ps.cM[s] = control_cm(ps.SM[s], ps.SO[s], ps.SP[s], ps.ratio, parabolic);
    }
  } else {
    // no downwind plane: linear control point
    ps.dsP = ps.kapP = ps.ikP = ps.tau0P = ps.ratio = 0.0;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      ps.SP[s] = 0.0;
      ps.cM[s] = 0.5 * (ps.SM[s] + ps.SO[s]);
    }
#pragma unroll
    for (int c = 0; c < 6; ++c) ps.epsP[c] = 0.0;
  }
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
  double dzM, dzP;   // |z_kO - z_kM|, |z_kP - z_kO|
  int ray0, nrb;     // rays [ray0, ray0 + nrb) of the enumeration
  T ibound;          // Stokes I on the boundary plane of this hemisphere
};

// ---------------------------------------------------------------------------
// Add the frequency-integrated Stokes vectors of a batch of rays on one plane to J^K_Q
// (Eq. 1) and Lbar, in a fixed order (no atomics).  A block takes kJNodes nodes; its
// threads are (ray group, node), group g summing rays g, g + G, ... over their frequency
// chunks, and the groups are added in order through LDS.  The loop over rays is a chain
// of memory latencies: with one thread per node and every ray in turn it took 25 us at
// 16x16 nodes and 40 rays, 73 us at 128x128 and 80 rays, more than the plane step that
// had to wait for it.  On the boundary plane the Stokes vector is (ibound, 0, 0, 0) at
// every frequency.  NS: Stokes parameters in the partial sums (4, or 1: intensity only).
// ---------------------------------------------------------------------------
constexpr int kJNodes = 16;   // consecutive nodes of a block: one 128-byte line of doubles
inline int jblocks(int np) { return (np + kJNodes - 1) / kJNodes; }
inline size_t jlds_bytes(int block) { return (size_t)block * 10 * sizeof(double); }

// acc += the projections of one ray's integrated Stokes vector.  T^K_Q is zero for
// Stokes V at K = 0, 2, for I, Q, U at K = 1, and for Q, U at J00 and U at J20.
template <int NS>
__device__ inline void jproject(const RayConsts& rc, const double ib[NS], double lam,
                                double acc[10]) {
  const double w = rc.weight;
  acc[0] += w * (rc.proj[0][0] * ib[0]);
  if constexpr (NS == 4) {
#pragma unroll
    for (int c = 1; c < 4; ++c) acc[c] += w * (rc.proj[c][3] * ib[3]);
    acc[4] += w * (rc.proj[4][0] * ib[0] + rc.proj[4][1] * ib[1]);
#pragma unroll
    for (int c = 5; c < 9; ++c)
      acc[c] += w * (rc.proj[c][0] * ib[0] + rc.proj[c][1] * ib[1] + rc.proj[c][2] * ib[2]);
  } else {
#pragma unroll
    for (int c = 4; c < 9; ++c) acc[c] += w * (rc.proj[c][0] * ib[0]);
  }
  acc[9] += w * lam;
}

template <int NS>
__device__ inline void jsum_rays(const double* __restrict__ jpart,
                                 const RayConsts* __restrict__ rays, int nrb, int nchunk, int np,
                                 int p, double ibound, double acc[10]) {
  const int g = threadIdx.x / kJNodes, G = blockDim.x / kJNodes;
  for (int rb = g; rb < nrb; rb += G) {
    double ib[NS], lam = 0.0;
#pragma unroll
    for (int s = 0; s < NS; ++s) ib[s] = 0.0;
    if (!jpart) {
      ib[0] = ibound;
    } else {
      const double* jp = jpart + (size_t)rb * nchunk * (NS + 1) * np + p;
#pragma unroll 4
      for (int c = 0; c < nchunk; ++c) {
#pragma unroll
        for (int s = 0; s < NS; ++s) ib[s] += jp[s * (size_t)np];
        lam += jp[NS * (size_t)np];
        jp += (NS + 1) * (size_t)np;
      }
    }
    jproject<NS>(rays[rb], ib, lam, acc);
  }
}

// lds: jlds_bytes(blockDim.x); every thread of the block calls it.
__device__ inline void jadd_groups(const double acc[10], double* __restrict__ jkq, size_t N,
                                   size_t plane_off, int np, int node0, double* lds) {
  const int n = threadIdx.x % kJNodes, g = threadIdx.x / kJNodes, G = blockDim.x / kJNodes;
#pragma unroll
  for (int c = 0; c < 10; ++c) lds[(c * G + g) * kJNodes + n] = acc[c];
  __syncthreads();
  for (int e = threadIdx.x; e < 10 * kJNodes; e += blockDim.x) {
    const int c = e / kJNodes, q = node0 + e % kJNodes;
    double sum = 0.0;
    for (int k = 0; k < G; ++k) sum += lds[(c * G + k) * kJNodes + e % kJNodes];
    if (q < np) jkq[c * N + plane_off + q] += sum;
  }
}

template <int NS>
__global__ void __launch_bounds__(256)
    k_jreduce(double* __restrict__ jkq, const double* __restrict__ jpart,
              const RayConsts* __restrict__ rays, int ray0, int nrb, int nchunk, int np, size_t N,
              size_t plane_off, double ibound) {
  extern __shared__ double s_tab[];
  const int node0 = blockIdx.x * kJNodes, p = node0 + threadIdx.x % kJNodes;
  double acc[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  if (p < np) jsum_rays<NS>(jpart, rays + ray0, nrb, nchunk, np, p, ibound, acc);
  jadd_groups(acc, jkq, N, plane_off, np, node0, s_tab);
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
  const T* phi;
  const double* wn;
  HemiArgs<T> h[2];
  double* jkq;       // [10][N] or nullptr
  size_t N;
  int nx, ny, np, nfreq;
  int ntile;         // tiles of blockDim.x nodes in a plane
  int nchunk, fchunk;
  int nstep;         // blocks of the plane step; the J reduction's follow
  int njb;           // blocks of the J reduction
  int jsame;         // both hemispheres' previous plane is the same one: one block adds both
  double inv_dx, inv_dy;
  int xcd_remap;     // tiles per XCD per round (0: hardware order), see xcd_tile
  int parabolic;     // control point: 0 BESSER, 1 parabola through M, O, P
};

// The arguments of one hemisphere, field by field: an index into a.h taken at run time
// would leave the pointers without their address space (flat loads and stores, 2% of
// the sweep at 256x256x128).
template <class T>
__device__ inline HemiArgs<T> hemi_args(const PlaneArgs<T>& a, bool second) {
  const HemiArgs<T>&u = a.h[0], &d = a.h[1];
  HemiArgs<T> h;
  h.iprev = second ? d.iprev : u.iprev;
  h.inext = second ? d.inext : u.inext;
  h.jpart = second ? d.jpart : u.jpart;
  h.jpart_prev = second ? d.jpart_prev : u.jpart_prev;
  h.prev_off = second ? d.prev_off : u.prev_off;
  h.kO = second ? d.kO : u.kO;
  h.kM = second ? d.kM : u.kM;
  h.kP = second ? d.kP : u.kP;
  h.dzM = second ? d.dzM : u.dzM;
  h.dzP = second ? d.dzP : u.dzP;
  h.ray0 = second ? d.ray0 : u.ray0;
  h.nrb = second ? d.nrb : u.nrb;
  h.ibound = second ? d.ibound : u.ibound;
  return h;
}

// The J reduction of the previous planes by the last njb blocks of a plane step: half of
// them for each hemisphere.
template <int NS, class T>
__device__ inline void jblock(const PlaneArgs<T>& a, double* lds) {
  const int b = blockIdx.x - a.nstep, per = a.njb / 2, hemi = b >= per;
  const int node0 = (b - hemi * per) * kJNodes;
  const HemiArgs<T> h = hemi_args(a, hemi);
  if (node0 >= a.np || h.nrb == 0 || (hemi && a.jsame)) return;
  const int p = node0 + threadIdx.x % kJNodes;
  double acc[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  if (p < a.np) {
    jsum_rays<NS>(h.jpart_prev, a.rays + h.ray0, h.nrb, a.nchunk, a.np, p, (double)h.ibound, acc);
    if (a.jsame)
      jsum_rays<NS>(a.h[1].jpart_prev, a.rays + a.h[1].ray0, a.h[1].nrb, a.nchunk, a.np, p,
                    (double)a.h[1].ibound, acc);
  }
  jadd_groups(acc, a.jkq, a.N, h.prev_off, a.np, node0, lds);
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

// The same over a two-dimensional grid of tiles.
__device__ inline void xcd_tile(int chunk, int& bx, int& by) {
  bx = blockIdx.x;
  by = blockIdx.y;
  if (chunk <= 0) return;
  const int Lp = xcd_order(chunk, blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
  bx = Lp % gridDim.x;
  by = Lp / gridDim.x;
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

constexpr int kMaxFreq = 4096;   // frequencies held in LDS by the sweep kernels

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
  setup_point<MODE>(a.kappa, a.prop, a.emis, a.N, a.nx, a.ny, a.np, h.kO, h.kM, h.kP, h.dzM,
                    h.dzP, a.inv_dx, a.inv_dy, rc, p, a.parabolic != 0, ps, sM9);
  const BezW<T> bwx = bez_weights(MODE == 1 ? (T)sM9.tx : T(0));
  const BezW<T> bwy = bez_weights(MODE == 1 ? (T)sM9.ty : T(0));
  const Stencil& sM = ps.sM;
  const double ikM = ps.ikM, ikO = ps.ikO;
  const double* etaM = ps.etaM;
  const double* etaO = ps.etaO;
  const double* SM = ps.SM;
  const double* SO = ps.SO;
  const double* cM = ps.cM;
  const double tau0M = ps.tau0M;
  // Lambda* = omega_O + omega_C c_M for a unit source at O alone (Eq. 14): c_M is 1 for
  // BESSER, (1 + ratio)/2 for the parabola, 1/2 without a downwind point
  const double lamfac = ps.hasP ? control_cm(0.0, 1.0, 0.0, ps.ratio, a.parabolic != 0) : 0.5;

  // frequency-independent pieces in the sweep precision
  const T eMv[3] = {(T)(etaM[0] * ikM), (T)(etaM[1] * ikM), (T)(etaM[2] * ikM)};
  const T rMv[3] = {(T)(etaM[3] * ikM), (T)(etaM[4] * ikM), (T)(etaM[5] * ikM)};
  const T eOv[3] = {(T)(etaO[0] * ikO), (T)(etaO[1] * ikO), (T)(etaO[2] * ikO)};
  const T rOv[3] = {(T)(etaO[3] * ikO), (T)(etaO[4] * ikO), (T)(etaO[5] * ikO)};
  const StokesOp<T> KO = stokes_op(eOv, rOv);
  T SMt[4], SOt[4], cMt[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    SMt[s] = (T)SM[s];
    SOt[s] = (T)SO[s];
    cMt[s] = (T)cM[s];
  }
  const T tau0 = (T)tau0M;
  const T w00 = (T)sM.w00, w10 = (T)sM.w10, w01 = (T)sM.w01, w11 = (T)sM.w11;
  const T lf = (T)lamfac;

  const size_t fstride = (size_t)a.np * 4;
  const size_t foff = ((size_t)sb.rb * a.nfreq + f0) * fstride;
  const T* ip = h.iprev ? h.iprev + foff : nullptr;
  T* op = h.inext + foff + (size_t)p * 4;
  double jacc0 = 0.0, jacc1 = 0.0, jacc2 = 0.0, jacc3 = 0.0, lacc = 0.0;

  // one update (Eq. fsbez solved with Eq. kappa) at frequency f0 + f from the upwind
  // Stokes vector IM
  auto update = [&](int f, T i0, T i1, T i2, T i3) __attribute__((always_inline)) {
    const T IM[4] = {i0, i1, i2, i3};
    const T tau = tau0 * s_phi[f];
    const Coefs<T> cf = coefficients(tau);
    T KI[4];
    kprime_apply(eMv, rMv, IM, KI);
    T b[4];
#pragma unroll
    for (int s = 0; s < 4; ++s)
      b[s] = fma_t(cf.omC, cMt[s], fma_t(cf.omO, SOt[s], fma_t(cf.omM, SMt[s],
                   fma_t(cf.e, IM[s], -(cf.psiM * KI[s])))));
    T x[4];
    stokes_solve<1>(KO, stokes_freq(KO, cf.psiO), b, x);
    store4_nt(op + (size_t)f * fstride, x);
    const double W = s_wn[f];
    jacc0 += W * (double)x[0];
    jacc1 += W * (double)x[1];
    jacc2 += W * (double)x[2];
    jacc3 += W * (double)x[3];
    lacc += W * (double)fma_t(lf, cf.omC, cf.omO);
  };
  // bilinear upwind component s from the four corner values
#define PORTA_BILIN(v, s) bilinear(w00, w10, w01, w11, v[0][s], v[1][s], v[2][s], v[3][s])

  if (!ip) {
    // the upwind plane is the boundary
    for (int f = 0; f < nf; ++f) update(f, h.ibound, T(0), T(0), T(0));
  } else if (MODE == 1) {
    for (int f = 0; f < nf; ++f) {
      T IM[4];
      upwind_bez9(ip + (size_t)f * fstride, sM9, bwx, bwy, IM);
      update(f, IM[0], IM[1], IM[2], IM[3]);
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
               PORTA_BILIN(vA, 3));
        load_upwind(ip + (size_t)min(f + 2, nf - 1) * fstride, sM, vA);
        update(f + 1, PORTA_BILIN(vB, 0), PORTA_BILIN(vB, 1), PORTA_BILIN(vB, 2),
               PORTA_BILIN(vB, 3));
      }
      if (f < nf)
        update(f, PORTA_BILIN(vA, 0), PORTA_BILIN(vA, 1), PORTA_BILIN(vA, 2),
               PORTA_BILIN(vA, 3));
    } else {
      T v[4][4];
      for (int f = 0; f < nf; ++f) {
        load_upwind(ip + (size_t)f * fstride, sM, v);
        update(f, PORTA_BILIN(v, 0), PORTA_BILIN(v, 1), PORTA_BILIN(v, 2), PORTA_BILIN(v, 3));
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
