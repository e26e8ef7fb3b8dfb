// porta_faces.hpp -- the plane step of the sweep with M and P on the first face of
// the grid that the short characteristic crosses (Sect. 3.1: M and P may lie on a
// vertical plane of the grid instead of a horizontal one).
//
// With uniform spacing in x and y the first face is of the same kind for every node
// of a plane, for a given ray: the horizontal plane next to it (within one cell),
// a vertical plane x = const through the neighbouring column, or y = const through
// the neighbouring row.  On a vertical face the point is interpolated bilinearly in
// (y, z) or (x, z) from two nodes of plane k itself and two of the upwind plane, so
// the nodes of plane k depend on each other along the ray's horizontal direction and,
// x and y being periodic, around the box.  The plane is then the fixed point of its
// node equations.  A block holds one ray and a few frequencies of a whole plane and
// marches across it row by row: each step solves one row of nodes (the lanes, at
// consecutive addresses) from the previous row (kept in LDS, in FP64 in either
// precision) and the upwind plane.  A
// ray that reaches an x = const face before a y = const one is solved on a transposed
// copy of the transfer coefficients (its own plane states transposed too), so that its
// in-plane dependencies also run from row to row.  The march starts m rows early: the
// part of I_M taken from plane k carries the weight 1 - t_z per
// step (t_z the fraction of the layer the ray descends while crossing a cell), and the
// rest of the update is a contraction, so after m >= ln(tol)/ln(1 - t_z) steps the
// starting guess no longer shows at the working precision and the remaining rows are
// the fixed point.  The frequency-independent work (interpolation of the transfer
// coefficients on the faces, S, K', control points, in FP64) is done once per node and
// ray by a parallel kernel before the march, which reads its results in the sweep
// precision as rows of a plane-sized table.
#pragma once

#include "porta_kernels.hpp"

namespace porta {

// The working frame of a ray: the grid as stored, or with x and y exchanged for a ray
// that meets a vertical face x = const before one y = const, so that in the working
// frame the first vertical face is always y = const (ties also go to y).
struct Frame {
  bool tr;                 // x and y exchanged
  int nx, ny;              // sizes in the working frame
  double inv_dx, inv_dy;
  double sx, sy;           // horizontal direction of the ray in the working frame
};

__device__ inline Frame ray_frame(const RayConsts& rc, int nx, int ny, double inv_dx,
                                  double inv_dy) {
  Frame f;
  f.tr = fabs(rc.sx) * inv_dx > fabs(rc.sy) * inv_dy;
  f.nx = f.tr ? ny : nx;
  f.ny = f.tr ? nx : ny;
  f.inv_dx = f.tr ? inv_dy : inv_dx;
  f.inv_dy = f.tr ? inv_dx : inv_dy;
  f.sx = f.tr ? rc.sy : rc.sx;
  f.sy = f.tr ? rc.sx : rc.sy;
  return f;
}

// First face crossed from a node, going upwind (dir = -1, point M) or downwind
// (dir = +1, point P), in the working frame: the plane next to it (kind 0) or the
// vertical plane y = const of the neighbouring row (kind 2), with the offsets and
// fractions of the bilinear interpolation on that face.  The path to the plane and the
// shift on it are formed as in setup_point, so that a horizontal face gives the
// plane-hop kernel's stencil.
struct FaceGeom {
  int kind;       // 0: horizontal plane kz; 2: y = const (row j + off)
  int off;        // +-1: the neighbouring row (kind 2)
  double ds;      // path length from O to the face
  double u, v;    // offsets of the point in cells (kind 0: both; kind 2: u)
  double tz;      // kind 2: fraction of the way from plane k to plane kz
};

__device__ inline FaceGeom face_geom(double mu, const Frame& fr, int dir, double dz) {
  const double inv_mu = 1.0 / fabs(mu);
  const double sz = dz * inv_mu;
  const double uy = dir * fr.sy;
  const double syf = uy != 0.0 ? 1.0 / (fabs(uy) * fr.inv_dy) : INFINITY;
  FaceGeom g;
  if (sz <= syf) {   // the frame puts the x face no nearer than the y face
    g.kind = 0;
    g.off = 0;
    g.ds = sz;
    g.u = dir * (sz * fr.sx * fr.inv_dx);
    g.v = dir * (sz * fr.sy * fr.inv_dy);
    g.tz = 1.0;
  } else {
    g.kind = 2;
    g.off = uy > 0.0 ? 1 : -1;
    g.ds = syf;
    g.u = syf * (dir * fr.sx) * fr.inv_dx;
    g.v = 0.0;
    g.tz = syf / sz;
  }
  return g;
}

// The four nodes and weights of a face point of node (i, j) of the working frame: on a
// horizontal face the bilinear stencil on plane kz; on a y face nodes 0, 1 on plane k
// (row j + off) and 2, 3 the same columns on plane kz.  Indices within a plane.
struct FaceStencil {
  int n[4];
  double w[4];
  double a, b;    // the same as two linear steps: a between nodes 0, 1 (and 2, 3), b from
                  // the pair 0, 1 to the pair 2, 3
  bool inplane;   // nodes 0 and 1 lie on plane k itself
};

__device__ inline FaceStencil face_stencil(const FaceGeom& g, int i, int j, int nx, int ny) {
  FaceStencil s;
  if (g.kind == 0) {
    const Stencil b = make_stencil(i, j, nx, ny, g.u, g.v);
    s.n[0] = b.i00; s.n[1] = b.i10; s.n[2] = b.i01; s.n[3] = b.i11;
    s.w[0] = b.w00; s.w[1] = b.w10; s.w[2] = b.w01; s.w[3] = b.w11;
    // the fractions of the cell, reduced as make_stencil reduces them
    const double u = g.u - nx * floor(g.u / nx), v = g.v - ny * floor(g.v / ny);
    s.a = u - floor(u);
    s.b = v - floor(v);
    s.inplane = false;
    return s;
  }
  s.inplane = true;
  const double fu = floor(g.u), f = g.u - fu;
  const int jc = wrapi(j + g.off, ny);
  const int i0 = wrapi(i + (int)fu, nx);
  // |u| <= 1, and at |u| = 1 (f = 0) the second corner has weight 0: take the first
  // again, so the corners of row j are always columns i - 1, i or i + 1
  const int i1 = f == 0.0 ? i0 : ((i0 + 1 == nx) ? 0 : i0 + 1);
  s.n[0] = jc * nx + i0; s.n[1] = jc * nx + i1;
  s.n[2] = s.n[0];       s.n[3] = s.n[1];
  s.w[0] = (1.0 - f) * (1.0 - g.tz);
  s.w[1] = f * (1.0 - g.tz);
  s.w[2] = (1.0 - f) * g.tz;
  s.w[3] = f * g.tz;
  s.a = f;
  s.b = g.tz;
  return s;
}

// A field at a face point: planes k (offset bk) and kz (offset bz).
template <class T>
__device__ inline double face_val(const T* __restrict__ f, const FaceStencil& s, size_t bk,
                                  size_t bz) {
  const size_t b01 = s.inplane ? bk : bz;
  return fma_t(s.w[3], (double)f[bz + s.n[3]],
               dot3(s.w[1], (double)f[b01 + s.n[1]], s.w[0], (double)f[b01 + s.n[0]], s.w[2],
                    (double)f[bz + s.n[2]]));
}

// One hemisphere's part of a launch: its plane, its rays and their states.
template <class T>
struct FacesHemi {
  const T* iprev;    // upwind plane states ([ray][freq][node][4], node in the ray's
                     // working frame), or nullptr: the boundary
  T* inext;          // states of plane kO, same layout
  int top;           // inext is I_top: nodes in the stored frame
  int kO, kM, kP;    // plane of O, upwind plane, downwind plane (-1: none)
  double dzM, dzP;
  int ray0, nrb;
  T ibound;
};

template <class T>
struct FacesArgs {
  const T* kappa;    // transfer coefficients as stored
  const T* prop;
  const T* emis;
  const T* kappa_t;  // the same with x and y exchanged in every plane
  const T* prop_t;
  const T* emis_t;
  const RayConsts* rays;
  const T* phi;
  const double* wn;
  FacesHemi<T> h[2]; // upward and downward rays, each on its own plane
  double* jchunk;    // [ray][chunk][5][node] (working frame): per frequency chunk,
                     // sum_j W_j I_i and sum_j W_j Lambda*, or nullptr
  T* cache;          // [ray][kFacesCache][node] (working frame): the set-up of each node
  size_t N;
  int nx, ny, np, nfreq, fchunk, nchunk;
  int lanes;         // columns of a block
  double inv_dx, inv_dy;
  int parabolic;
  double tol;        // the march's starting guess is damped below tol (the unit roundoff)
  int nrb;           // rays of the launch, the upward ones first
};

// Field by field, as hemi_args.
template <class T>
__device__ inline FacesHemi<T> faces_hemi(const FacesArgs<T>& a, bool second) {
  const FacesHemi<T>&u = a.h[0], &d = a.h[1];
  FacesHemi<T> h;
  h.iprev = second ? d.iprev : u.iprev;
  h.inext = second ? d.inext : u.inext;
  h.top = second ? d.top : u.top;
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

// Workgroups of a launch go to the 8 XCDs in turn (workgroup w to XCD w % 8).  The march
// takes a one-dimensional grid of 8 * ceil(nrb / 8) * nchunk workgroups and gives XCD x
// the rays x, x + 8, x + 16, ... (every inclination alike on each XCD), each ray's
// chunks one after another: they start together and walk the same rows, so the rows
// of the set-up table that every chunk of the ray reads come from that XCD's L2.
constexpr int kFacesXcds = 8;
inline int faces_grid(int nrb, int nchunk) {
  return kFacesXcds * ((nrb + kFacesXcds - 1) / kFacesXcds) * nchunk;
}

// Values of the set-up of a node and ray that the march reads, in the sweep precision:
// K'_M / eta_I entries (eta 3, rho 3), K'_O (3, 3), the three source values of I, Q and U
// (StepSource), the optical depth tau_MO at line centre and the Lambda* factor of omega_C.
enum FacesCacheSlot {
  kCeM = 0, kCrM = 3, kCeO = 6, kCrO = 9, kCSa = 12, kCSb = 15, kCSc = 18, kCtau = 21,
  kClf = 22, kFacesCache = 23
};

// How the march of a launch is cut: a block holds one ray, `lanes` columns and fchunk
// frequencies; its threads are (column, one of `ways` sets of the chunk's frequencies), and a
// thread carries the fchunk / ways frequencies of its set.
//
// A march is a serial chain of rows (up to 17 / t_z of them in FP32 for the most inclined
// rays), so on small planes its length is what counts: every thread takes one frequency and
// the blocks are those that share the partial sums of J.  Once there are more wavefronts
// than the chip holds, threads take several frequencies: the row's set-up is then read once
// for all of them.  At 256x256x128, 80 rays and 101 frequencies, with one set per block, a
// sweep took 2.53 and 2.59 s with 4 and 5 frequencies a thread in FP32; 6.51, 6.49 and 6.37 s
// with 5, 6 and 7 in FP64.
template <class T>
__host__ __device__ constexpr int faces_serial() {   // frequencies of a thread, at most
  return sizeof(T) == 4 ? 4 : 7;
}
template <class T>
__host__ __device__ constexpr int faces_waves() {    // wavefronts that the chip holds
  return 1024 * (sizeof(T) == 4 ? 4 : 2);
}
constexpr int kFacesMaxLanes = 512;  // columns of a plane held by one block
constexpr int kFacesThreads = 512;   // threads of a block, at most
constexpr int kFacesMaxWays = 8;
constexpr int kFacesMaxWarm = 65536; // warm-up rows of a march, at most
constexpr size_t kFacesLds = 65536;  // LDS of one block, at most

// LDS of the kernel: W_j and phi_j of the chunk's frequencies; then (16-byte aligned) the row
// of Stokes vectors of each lane, [f][lane][4]; then the first and last lane's vectors of
// every wave, twice (rows of even and odd parity), [parity][f][wave][2][4]; then, with
// several ways, their partial sums of J for rows of either parity, [parity][way][5][lane].
// The previous row's Stokes vectors are kept in FP64 in either precision (see
// k_sweep_plane_faces).
template <class T>
__host__ __device__ inline size_t faces_col_offset(int fchunk) {
  return ((size_t)fchunk * (sizeof(double) + sizeof(T)) + 15) & ~(size_t)15;
}
template <class T>
__host__ __device__ inline size_t faces_lds_bytes(int fchunk, int lanes, int ways) {
  const size_t waves = (size_t)(lanes + 63) / 64;
  return faces_col_offset<T>(fchunk) + (size_t)fchunk * (lanes + 4 * waves) * 4 * sizeof(double) +
         (ways > 1 ? (size_t)2 * ways * 5 * lanes * sizeof(double) : 0);
}

// Frequency-independent part of the update of node p (working frame): the PointSetup of
// the plane-hop kernel with the coefficients at M and P taken on their faces.
template <class T>
__device__ inline void setup_point_faces(const T* __restrict__ kappa, const T* __restrict__ prop,
                                         const T* __restrict__ emis, const FacesArgs<T>& a,
                                         const FacesHemi<T>& h, const RayConsts& rc, const FaceGeom& gM,
                                         const FaceStencil& sM, const FaceGeom& gP,
                                         const FaceStencil& sP, bool hasP, int p,
                                         PointSetup& ps) {
  const size_t N = a.N, bk = (size_t)h.kO * a.np, bM = (size_t)h.kM * a.np;
  ps.dsM = gM.ds;
  ps.kapM = face_val(kappa, sM, bk, bM);
#pragma unroll
  for (int c = 0; c < 6; ++c) {
    ps.epsM[c] = face_val(emis + c * N, sM, bk, bM);
    ps.etaM[c] = face_val(prop + c * N, sM, bk, bM);
  }
  const size_t bO = bk + p;
  ps.kapO = (double)kappa[bO];
#pragma unroll
  for (int c = 0; c < 6; ++c) {
    ps.epsO[c] = (double)emis[c * N + bO];
    ps.etaO[c] = (double)prop[c * N + bO];
  }
  ps.hasP = hasP;
  if (hasP) {
    const size_t bP = (size_t)h.kP * a.np;
    ps.dsP = gP.ds;
    ps.kapP = face_val(kappa, sP, bk, bP);
#pragma unroll
    for (int c = 0; c < 6; ++c) ps.epsP[c] = face_val(emis + c * N, sP, bk, bP);
  }
  setup_sources(rc, a.parabolic != 0, ps);
}

// The frequency-independent set-up of every node of plane kO (working frame) for every
// ray of the batch (blockIdx.y), in FP64, stored in the sweep precision.
template <class T>
__global__ void __launch_bounds__(256) k_faces_setup(const FacesArgs<T> a) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x, rb = blockIdx.y;
  if (p >= a.np) return;
  const bool down = rb >= a.h[0].nrb;
  const FacesHemi<T> h = faces_hemi(a, down);
  const RayConsts& rc = a.rays[h.ray0 + rb - (down ? a.h[0].nrb : 0)];
  const Frame fr = ray_frame(rc, a.nx, a.ny, a.inv_dx, a.inv_dy);
  const T* kappa = fr.tr ? a.kappa_t : a.kappa;
  const T* prop = fr.tr ? a.prop_t : a.prop;
  const T* emis = fr.tr ? a.emis_t : a.emis;
  const FaceGeom gM = face_geom(rc.mu, fr, -1, h.dzM);
  const bool hasP = h.kP >= 0;
  const FaceGeom gP = hasP ? face_geom(rc.mu, fr, +1, h.dzP) : gM;
  const int i = p % fr.nx, j = p / fr.nx;
  const FaceStencil sM = face_stencil(gM, i, j, fr.nx, fr.ny);
  const FaceStencil sP = hasP ? face_stencil(gP, i, j, fr.nx, fr.ny) : sM;
  PointSetup ps;
  setup_point_faces(kappa, prop, emis, a, h, rc, gM, sM, gP, sP, hasP, p, ps);
  const size_t np = (size_t)a.np;
  T* c = a.cache + (size_t)rb * kFacesCache * np + p;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    c[(kCeM + k) * np] = (T)(ps.etaM[k] * ps.ikM);
    c[(kCrM + k) * np] = (T)(ps.etaM[3 + k] * ps.ikM);
    c[(kCeO + k) * np] = (T)(ps.etaO[k] * ps.ikO);
    c[(kCrO + k) * np] = (T)(ps.etaO[3 + k] * ps.ikO);
  }
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    StepSource<T> t;
    step_source(ps.SM[s], ps.SO[s], ps.cM[s], t);
    c[(kCSa + s) * np] = t.a;
    c[(kCSb + s) * np] = t.b;
    c[(kCSc + s) * np] = t.c;
  }
  c[kCtau * np] = (T)ps.tau0M;
  c[kClf * np] = (T)ps.lamfac;
}

// The set-up of one node and ray as the march reads it.
template <class T>
struct FacesNode {
  T eM[3], rM[3], eO[3], rO[3];
  StepSource<T> src[3];
  T tau0, lf;
};

template <class T>
__device__ inline void load_node(const T* __restrict__ cp, size_t np, FacesNode<T>& n) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    n.eM[k] = cp[(kCeM + k) * np];
    n.rM[k] = cp[(kCrM + k) * np];
    n.eO[k] = cp[(kCeO + k) * np];
    n.rO[k] = cp[(kCrO + k) * np];
    n.src[k] = {cp[(kCSa + k) * np], cp[(kCSb + k) * np], cp[(kCSc + k) * np]};
  }
  n.tau0 = cp[kCtau * np];
  n.lf = cp[kClf * np];
}

// One plane for one ray and one chunk of frequencies (order: faces_grid).  The lanes of a
// wavefront are columns of the working frame; the block walks its rows.  Each thread keeps
// its own column's Stokes vectors of the previous row in LDS (FP64) and reads the neighbouring
// column's there too when that lane is in its wave (the lanes of a wave read before
// they write); a neighbour in another wave is read from the copy of the first and last
// lanes of every wave, which is kept for rows of either parity, so one barrier per row
// orders the exchange.  A ray whose first face is the plane itself has no in-plane
// dependency, and columns that fit in one wavefront exchange nothing between waves: they
// take no barrier but the one that the sum of J over the ways needs on stored rows.
//
// ONE: a thread carries one frequency.  It then loads the next row's upwind corners, and in
// FP32 its set-up (in FP64 that spills), during the current one: their wait was most of a
// row's time.  64x64x64, 40 rays a hemisphere, 41 frequencies in FP32: a plane of both
// hemispheres in 914 us, with blocks of one wavefront, 4 frequencies in turn, no loads ahead
// and a launch per hemisphere 2 x 1289 us.  What bounds it is the latency of a row (LDS
// exchange, 4x4 solve), for 64 columns about 2 wavefronts on each SIMD.
template <class T, bool ONE>
__global__ void __launch_bounds__(kFacesThreads)
__attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 2 : (ONE ? 3 : 4))))
k_sweep_plane_faces(const FacesArgs<T> a) {
  constexpr bool AHEAD = ONE && sizeof(T) == 4;   // the set-up too is loaded a row ahead
  // this workgroup's ray and chunk (faces_grid); the few past the last ray leave at once
  const int wx = blockIdx.x % kFacesXcds, wk = blockIdx.x / kFacesXcds;
  const int rb = wx + kFacesXcds * (wk / a.nchunk), chunk = wk % a.nchunk;
  if (rb >= a.nrb) return;
  const bool down = rb >= a.h[0].nrb;
  const FacesHemi<T> h = faces_hemi(a, down);
  const int hrb = rb - (down ? a.h[0].nrb : 0);   // ray within its hemisphere
  extern __shared__ double s_tab[];
  double* s_wn = s_tab;
  T* s_phi = reinterpret_cast<T*>(s_tab + a.fchunk);
  // the in-plane chain in FP64 (D): on the thin cell steps of an inclined ray in the line
  // wings the change of I per step falls below half a unit in the last place of an FP32
  // I, so an FP32 chain would drop it at every step; the FP32 arithmetic forms that
  // change and the chain adds it in FP64 (the plane states stored are FP32)
  using D = double;
  D* s_row = reinterpret_cast<D*>(reinterpret_cast<char*>(s_tab) + faces_col_offset<T>(a.fchunk));
  const int lanes = a.lanes, nwaves = lanes >> 6, ways = blockDim.x / lanes;
  D* s_bnd = s_row + (size_t)a.fchunk * lanes * 4;
  const size_t bpar = (size_t)a.fchunk * nwaves * 8;   // one parity of s_bnd
  D* s_red = s_bnd + 2 * bpar;
  const int f0 = chunk * a.fchunk;
  const int nf = min(a.fchunk, a.nfreq - f0);
  for (int t = threadIdx.x; t < nf; t += blockDim.x) {
    s_wn[t] = a.wn[f0 + t];
    s_phi[t] = a.phi[f0 + t];
  }
  const RayConsts& rc = a.rays[h.ray0 + hrb];
  const Frame fr = ray_frame(rc, a.nx, a.ny, a.inv_dx, a.inv_dy);
  const FaceGeom gM = face_geom(rc.mu, fr, -1, h.dzM);
  const bool chain = gM.kind != 0;   // same for the whole block
  const bool row_sync = chain && nwaves > 1;
  const size_t np = (size_t)a.np;
  const T* cache = a.cache + (size_t)rb * kFacesCache * np;
  const int lane = threadIdx.x % lanes, way = threadIdx.x / lanes, wave = lane >> 6;
  const bool active = lane < fr.nx;
  const int nstep = fr.ny;
  // march direction: away from the row M lies on (kind 0: any order)
  const int mdir = chain ? -gM.off : 1;
  int warm = 0;
  if (chain) {
    // (1 - t_z)^warm <= tol (37 / t_z rows in FP64, 17 / t_z in FP32), however many
    // times around the box that takes; at most kFacesMaxWarm rows (t_z >= 5.6e-4 in
    // FP64), clamped before the cast
    const double q = log1p(-fmin(gM.tz, 1.0));
    const double w = q < 0.0 ? ceil(log(a.tol) / q) : 0.0;
    warm = (int)fmin(fmax(w, 0.0), (double)kFacesMaxWarm);
  }
  const size_t fstride = (size_t)a.np * 4;
  const size_t foff = ((size_t)hrb * a.nfreq + f0) * fstride;
  const T* ip = h.iprev ? h.iprev + foff : nullptr;
  T* op = h.inext + foff;
  // this lane's slots: its own column, and its copy for the other waves if it is the
  // first or last active lane of its wave
  const int side = lane == (wave << 6) ? 0 : (lane == min((wave << 6) + 63, fr.nx - 1) ? 1 : -1);
  const bool last_too = side == 0 && lane == min((wave << 6) + 63, fr.nx - 1);
  // columns of the corners, and the rows of the two pairs relative to the node's: the same
  // for every row
  int ca = 0, cb = 0, ra = 0, rz = 0;
  double fa = 0.0, fb = 0.0;   // I_M as two linear steps, see below
  // where the two in-plane corners of the previous row are read (y face): the column's
  // own slot if its lane is in this wave, else the other wave's copy, whose offset
  // moves by bpar with the row's parity (corner = column i - 1, i or i + 1)
  int c_off[2] = {0, 0}, c_str[2] = {4 * lanes, 4 * lanes};
  bool c_bnd[2] = {false, false};
  if (active) {
    const FaceStencil s0 = face_stencil(gM, lane, 0, fr.nx, fr.ny);
    ca = s0.n[2] % fr.nx;
    cb = s0.n[3] % fr.nx;
    ra = s0.n[0] / fr.nx;
    rz = s0.n[2] / fr.nx;
    fa = s0.a;
    fb = s0.b;
    if (chain) {
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int l = c == 0 ? ca : cb, w = l >> 6;
        if (w == wave) {
          c_off[c] = 4 * l;
        } else {
          c_bnd[c] = true;
          c_str[c] = 8 * nwaves;
          c_off[c] = 8 * w + 4 * (l == (w << 6) ? 0 : 1);
        }
      }
    }
  }
  // the row before the first step: the upwind plane's values there (the guess)
  const int c_first = wrapi((mdir > 0 ? 0 : nstep - 1) - mdir * warm, nstep);
  if (chain) {
    const int cprev = wrapi(c_first - mdir, nstep);
    for (int f = way; f < nf && active; f += ways) {
      T v[4] = {h.ibound, T(0), T(0), T(0)};
      if (ip) load4(ip + (size_t)f * fstride + 4 * (size_t)(cprev * fr.nx + lane), v);
      const D vd[4] = {(D)v[0], (D)v[1], (D)v[2], (D)v[3]};
      store4(s_row + ((size_t)f * lanes + lane) * 4, vd);
      // the parity read at step 0 is that of step -1
      D* b = s_bnd + bpar + ((size_t)f * nwaves + wave) * 8;
      if (side >= 0) store4(b + 4 * side, vd);
      if (last_too) store4(b + 4, vd);
    }
  }
  __syncthreads();
  // the corners on the upwind plane of row j for frequency f: the pair that a y face takes
  // there, or both pairs of a horizontal face
  struct Upwind {
    T z[2][4], o[2][4];
  };
  auto load_up = [&](int j, int f, Upwind& u) __attribute__((always_inline)) {
    if (!ip) {
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        u.z[c][0] = u.o[c][0] = h.ibound;
#pragma unroll
        for (int s = 1; s < 4; ++s) u.z[c][s] = u.o[c][s] = T(0);
      }
      return;
    }
    const T* q = ip + (size_t)f * fstride;
    const size_t rowz = (size_t)shift_index(j, rz, nstep) * fr.nx;
    load4(q + 4 * (rowz + ca), u.z[0]);
    load4(q + 4 * (rowz + cb), u.z[1]);
    if (!chain) {
      const size_t rowa = (size_t)shift_index(j, ra, nstep) * fr.nx;
      load4(q + 4 * (rowa + ca), u.o[0]);
      load4(q + 4 * (rowa + cb), u.o[1]);
    }
  };
  double* jc = a.jchunk ? a.jchunk + ((size_t)rb * a.nchunk + chunk) * 5 * a.np : nullptr;
  FacesNode<T> node, node_next;
  Upwind up, up_next;
  const int total = warm + nstep;
  int j = c_first;
  if (ONE && active && way < nf) {
    if constexpr (AHEAD) load_node(cache + (size_t)j * fr.nx + lane, np, node);
    load_up(j, way, up);
  }
  for (int t = 0; t < total; ++t) {
    const int jn = mdir > 0 ? (j + 1 == nstep ? 0 : j + 1) : (j == 0 ? nstep - 1 : j - 1);
    const bool store = t >= warm;
    const size_t rd = (t & 1) ? 0 : bpar, wr = (t & 1) ? bpar : 0;   // s_bnd parities
    double jacc[4] = {0, 0, 0, 0}, lacc = 0.0;
    const int p = j * fr.nx + lane;                                   // working frame
    if (active && way < nf) {
      // (loads ahead of the last row: a row's are loaded once more and not used)
      if constexpr (AHEAD) load_node(cache + (size_t)jn * fr.nx + lane, np, node_next);
      else load_node(cache + p, np, node);
      if constexpr (ONE) load_up(jn, way, up_next);
      const auto KO = step_op(node.eO, node.rO);
      const D* r0 = (c_bnd[0] ? s_bnd + rd : s_row) + c_off[0];
      const D* r1 = (c_bnd[1] ? s_bnd + rd : s_row) + c_off[1];
      D* own = s_row + 4 * (size_t)lane;
      D* bown = s_bnd + wr + 8 * (size_t)wave;
      const size_t ostore = h.top && fr.tr ? (size_t)lane * a.nx + j : (size_t)p;   // stored frame
      for (int f = way; f < nf; f += ways) {
        if constexpr (!ONE) load_up(j, f, up);
        // I_M as two linear steps (x, then z or y): a field constant over the stencil is
        // returned exactly, so the rounding of the four weights, the same for every node
        // of a ray, adds no bias that the many cell steps of an inclined ray would pile up
        D IM[4];
        D c0[4], c1[4];
        if (chain) {
          load4(r0 + (size_t)f * c_str[0], c0);
          load4(r1 + (size_t)f * c_str[1], c1);
        } else {
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            c0[s] = up.o[0][s];
            c1[s] = up.o[1][s];
          }
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const D A = c0[s] + fa * (c1[s] - c0[s]);
          const D u0 = up.z[0][s], u1 = up.z[1][s];
          const D B = u0 + fa * (u1 - u0);
          IM[s] = A + fb * (B - A);
        }
        const Coefs<T> cf = coefficients(node.tau0 * s_phi[f]);
        const T IMt[4] = {(T)IM[0], (T)IM[1], (T)IM[2], (T)IM[3]};
        T KI[4], dv[4];
        kprime_apply<1, true>(node.eM, node.rM, IMt, KI);
        // e I_M as I_M - (1 - e) I_M (see Coefs::em1), and the change of a step summed
        // before it is added to I_M: on thin steps each term alone can fall below half
        // a unit in the last place of I_M, and dropping the source terms while keeping
        // the attenuation would bias a long chain of steps
        const StepSource<T> w = source_weights(cf);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          dv[s] = fma_t(-cf.em1, IMt[s], -(cf.psiM * KI[s]));
          if (s < 3) dv[s] = add_sources(w, node.src[s], dv[s]);
        }
        const auto F = step_freq(KO, cf.psiO);
        D res[4];
        if constexpr (sizeof(T) == 4) {
          // (1 + psi'_O K'_O) I_O = I_M + d, so I_O = I_M + x with
          // (1 + psi'_O K'_O) x = d - psi'_O K'_O I_M: x in FP32, I_M + x in FP64
          T KOI[4], rhs[4], x[4];
          kprime_apply<1, true>(node.eO, node.rO, IMt, KOI);
#pragma unroll
          for (int s = 0; s < 4; ++s) rhs[s] = fma_t(-cf.psiO, KOI[s], dv[s]);
          stokes_solve<1>(KO, F, rhs, x, true);
#pragma unroll
          for (int s = 0; s < 4; ++s) res[s] = IM[s] + (D)x[s];
        } else {
          T b[4];
#pragma unroll
          for (int s = 0; s < 4; ++s) b[s] = IM[s] + dv[s];
          stokes_solve<1>(KO, F, b, res);
        }
        if (chain) {
          store4(own + (size_t)f * lanes * 4, res);
          if (row_sync) {
            D* b2 = bown + (size_t)f * nwaves * 8;
            if (side >= 0) store4(b2 + 4 * side, res);
            if (last_too) store4(b2 + 4, res);
          }
        }
        if (store) {
          const T rest[4] = {(T)res[0], (T)res[1], (T)res[2], (T)res[3]};
          // I_top of a ray in the exchanged frame goes to the grid's own indices, across
          // rows: there the plain store, whose lines the cache merges, is the faster
          if (h.top) store4(op + (size_t)f * fstride + 4 * ostore, rest);
          else store4_nt(op + (size_t)f * fstride + 4 * ostore, rest);
          const double W = s_wn[f];
#pragma unroll
          for (int s = 0; s < 4; ++s) jacc[s] = fma_t(W, (double)res[s], jacc[s]);
          lacc = fma_t(W, (double)lambda_star(cf, node.lf), lacc);
        }
      }
      if constexpr (AHEAD) node = node_next;
      if constexpr (ONE) up = up_next;
    }
    if (store && jc) {
      const double v[5] = {jacc[0], jacc[1], jacc[2], jacc[3], lacc};
      if (ways == 1) {
        if (active)
#pragma unroll
          for (int c = 0; c < 5; ++c) __builtin_nontemporal_store(v[c], jc + c * np + p);
      } else {
        D* red = s_red + (size_t)(t & 1) * ways * 5 * lanes;
#pragma unroll
        for (int c = 0; c < 5; ++c) red[((size_t)way * 5 + c) * lanes + lane] = v[c];
        __syncthreads();
        if (active)
          for (int c = way; c < 5; c += ways) {
            double sum = 0.0;
            for (int k = 0; k < ways; ++k) sum += red[((size_t)k * 5 + c) * lanes + lane];
            __builtin_nontemporal_store(sum, jc + c * np + p);
          }
      }
    }
    // the row is complete (and its copies for the other waves) before the next reads it; the
    // barrier of the J sum, where there is one, comes after the writes to LDS above
    if (row_sync && !(store && jc && ways > 1)) __syncthreads();
    j = jn;
  }
}

// Transpose every plane of nfield fields ([field][k][ny][nx] -> [field][k][nx][ny]).
template <class T>
__global__ void __launch_bounds__(256)
    k_transpose_planes(const T* __restrict__ src, T* __restrict__ dst, int nx, int ny,
                       size_t nplanes) {
  const size_t np = (size_t)nx * ny;
  const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= np * nplanes) return;
  const size_t q = e / np, r = e % np;
  const int j = (int)(r % ny), i = (int)(r / ny);   // dst index r = i * ny + j
  dst[e] = src[q * np + (size_t)j * nx + i];
}

// Sum the frequency-chunk partials of every ray into the per-ray layout of the J
// reduction, from the ray's working frame to the grid's own: jpart[ray][5][node] =
// sum_chunk jchunk[ray][chunk][5][working node].  A block takes a 32 x 32 tile of the
// working frame (blockIdx.x, blockIdx.y over a square of the larger side) for one ray and
// component (blockIdx.z = 5 ray + component) and writes it through LDS, so that both the reads and, for a ray
// solved with x and y exchanged, the transposed writes are coalesced.
constexpr int kSumTile = 32;

__global__ void __launch_bounds__(256)
    k_sum_chunks(double* __restrict__ jpart, const double* __restrict__ jchunk,
                 const RayConsts* __restrict__ rays, int ray0, int nup, int ray1, int nchunk,
                 int nx, int ny, double inv_dx, double inv_dy) {
  __shared__ double tile[kSumTile][kSumTile + 1];
  const int rb = blockIdx.z / 5, c = blockIdx.z % 5;
  const Frame fr = ray_frame(rays[rb < nup ? ray0 + rb : ray1 + rb - nup], nx, ny, inv_dx, inv_dy);
  const int x0 = blockIdx.x * kSumTile, y0 = blockIdx.y * kSumTile;
  if (x0 >= fr.nx || y0 >= fr.ny) return;   // the same for the whole block
  const size_t np = (size_t)nx * ny;
  const int tx = threadIdx.x % kSumTile, ty = threadIdx.x / kSumTile;   // 32 x 8
  for (int r = ty; r < kSumTile; r += 8) {
    const int xw = x0 + tx, yw = y0 + r;
    double sum = 0.0;
    if (xw < fr.nx && yw < fr.ny) {
      const size_t pw = (size_t)yw * fr.nx + xw;
      const double* src = jchunk + ((size_t)rb * nchunk * 5 + c) * np + pw;
      const size_t kst = 5 * np;   // from one chunk to the next
      int k = 0;
      // eight loads in flight, then added in chunk order (the sum of one loop)
      for (; k + 8 <= nchunk; k += 8) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = src[(size_t)(k + u) * kst];
#pragma unroll
        for (int u = 0; u < 8; ++u) sum += v[u];
      }
      for (; k < nchunk; ++k) sum += src[(size_t)k * kst];
    }
    tile[r][tx] = sum;
  }
  __syncthreads();
  double* out = jpart + ((size_t)rb * 5 + c) * np;
  for (int r = ty; r < kSumTile; r += 8) {
    if (!fr.tr) {
      const int xw = x0 + tx, yw = y0 + r;
      if (xw < fr.nx && yw < fr.ny) out[(size_t)yw * nx + xw] = tile[r][tx];
    } else {
      // stored (x, y) = working (y, x): consecutive lanes take consecutive stored x
      const int yw = y0 + tx, xw = x0 + r;
      if (xw < fr.nx && yw < fr.ny) out[(size_t)xw * nx + yw] = tile[tx][r];
    }
  }
}

}  // namespace porta
