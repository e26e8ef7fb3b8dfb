// porta_pair.hpp -- two consecutive planes of the sweep in one launch.
//
// The plane-by-plane sweep moves every plane state through HBM twice, written by one launch
// and read by the next: 32 bytes per update in FP32, 64 in FP64, and at the sizes where
// it matters that is what bounds it.  Here a block solves a tile of the first plane, hands
// it to the second plane's update through LDS, and only the second plane's state goes to
// memory (the first plane's too where it is kept for the adjoint).  For a ray the points M of
// a plane are displaced by the same number of cells at every node, so the tile of the second
// plane needs a tile of the first that is one node wider and higher, shifted, and that one a
// tile of the upwind plane one wider and higher again; the rim nodes are solved by
// both neighbours, with the same result.
//
// A block has two groups of four wavefronts, one per plane, so that a thread holds the set-up
// of one node only.  At step f the first group solves frequency f from the upwind tile, the
// second frequency f - 1 from the first plane's tile, and the upwind tile of frequency f + 2
// is on its way from memory (one node per thread); one barrier per step orders the exchange.
#pragma once

#include "porta_kernels.hpp"

namespace porta {

constexpr int kPairGroup = 256;                 // threads of a group
constexpr int kPairThreads = 2 * kPairGroup;

// The tile of the second plane: 16 nodes wide, so that its stores are whole 128-byte lines,
// and as many rows as keep the first plane's tile (17 x 15) within a group.
constexpr int kPairX = 16, kPairY = 14;
constexpr int kMidX = kPairX + 1, kMidY = kPairY + 1;   // first plane
constexpr int kUpX = kPairX + 2, kUpY = kPairY + 2;     // upwind plane
static_assert(kMidX * kMidY <= kPairGroup && kUpX * kUpY <= kPairThreads, "tiles fit the groups");

inline int pair_tiles(int nx, int ny) {
  return ((nx - 1) / kPairX + 1) * ((ny - 1) / kPairY + 1);
}

// Partial sums of J of one earlier plane.
struct JPrev {
  const double* part;   // nullptr: the boundary plane
  size_t off;           // of the plane in jkq
};

// Whether a launch can hold both hemispheres, for sweeps whose one does not fill the chip: in
// FP64.  In FP32 the choice costs scalar registers and gains nothing over a plane of both per
// launch (64x64x49, 40 rays each, 31 frequencies: 3.8 ms either way).
template <class T>
constexpr bool kPairBoth = sizeof(T) == 8;

template <class T>
struct PairArgs {
  PlaneArgs<T> a;      // h[m]: the first plane of a hemisphere (inext: nullptr unless kept; not
                       // kPairBoth: h[0] is the launch's only one); jsame: both hemispheres add
                       // partial sums to the same plane of J
  HemiArgs<T> n[2];    // the second planes (iprev unused)
  JPrev jp[2][2];      // planes of the previous launch whose partial sums this one adds to J
  int njprev[2];       // how many of each hemisphere
  int ntx;             // tiles in a row of tiles
};

// A tile of Stokes vectors in LDS.  FP64 vectors are split into two arrays of pairs, so that
// neighbouring lanes read neighbouring 16 bytes.
template <class T, int N>
struct TileBuf;
template <int N>
struct TileBuf<float, N> {
  float4 v[N];
  __device__ void put(int i, const float x[4]) { v[i] = make_float4(x[0], x[1], x[2], x[3]); }
  __device__ void get(int i, float x[4]) const {
    const float4 q = v[i];
    x[0] = q.x; x[1] = q.y; x[2] = q.z; x[3] = q.w;
  }
};
template <int N>
struct TileBuf<double, N> {
  double2 a[N], b[N];
  __device__ void put(int i, const double x[4]) {
    a[i] = make_double2(x[0], x[1]);
    b[i] = make_double2(x[2], x[3]);
  }
  __device__ void get(int i, double x[4]) const {
    const double2 p = a[i], q = b[i];
    x[0] = p.x; x[1] = p.y; x[2] = q.x; x[3] = q.y;
  }
};

template <class T>
struct PairLds {
  TileBuf<T, kUpX * kUpY> up[2];
  TileBuf<T, kMidX * kMidY> mid[2];
};

// Bounded by its arithmetic and LDS reads at 4 wavefronts per SIMD in FP32, 2 in FP64 (the
// registers of a node's set-up).  A sweep of 256x256x128, 160 rays, 101 frequencies in FP32 takes
// 738 ms, plane by plane 845; one of 128x128x96, 160 rays, 41 frequencies in FP64 133.6 and 161.8.
template <class T>
__global__ void __launch_bounds__(kPairThreads)
__attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 2, sizeof(T) == 4 ? 4 : 2)))
k_sweep_pair(const PairArgs<T> A) {
  const PlaneArgs<T>& a = A.a;
  extern __shared__ double s_tab[];
  if ((int)blockIdx.x >= a.nstep) {
    // jblocks of them for each hemisphere and plane; where both hemispheres add to a plane, the
    // first jblocks do everything in turn.  The second half of the threads only synchronises.
    if constexpr (!kPairBoth<T>) {
      const int b = blockIdx.x - a.nstep, per = a.njb / 2, second = b >= per;
      if (second && A.njprev[0] < 2) return;
      const JJob j = {second ? A.jp[0][1].part : A.jp[0][0].part, a.rays + a.h[0].ray0, a.h[0].nrb,
                      1, (double)a.h[0].ibound, second ? A.jp[0][1].off : A.jp[0][0].off};
      jreduce_block<4, T>(j, a.jkq, a.N, a.np, (b - second * per) * kJNodes, s_tab, kPairGroup);
      return;
    }
    const int b = blockIdx.x - a.nstep, per = a.njb / 4, first = b / per;
    const int node0 = (b - first * per) * kJNodes;
    if (a.jsame && first > 0) return;
    for (int e = first; e < (a.jsame ? 4 : first + 1); ++e) {
      const bool down = e >= 2, second = e & 1;
      const HemiArgs<T> h = hemi_args(a, down);
      if (h.nrb == 0 || second >= (down ? A.njprev[1] : A.njprev[0])) continue;
      const double* up_part = second ? A.jp[0][1].part : A.jp[0][0].part;
      const double* down_part = second ? A.jp[1][1].part : A.jp[1][0].part;
      const size_t up_off = second ? A.jp[0][1].off : A.jp[0][0].off;
      const size_t down_off = second ? A.jp[1][1].off : A.jp[1][0].off;
      const JJob j = {down ? down_part : up_part, a.rays + h.ray0, h.nrb, 1, (double)h.ibound,
                      down ? down_off : up_off};
      __syncthreads();   // the last one's LDS has been read
      jreduce_block<4, T>(j, a.jkq, a.N, a.np, node0, s_tab, kPairGroup);
    }
    return;
  }
  __shared__ PairLds<T> lds;
  double* s_wn = s_tab;
  T* s_phi = reinterpret_cast<T*>(s_tab + a.nfreq);
  for (int t = threadIdx.x; t < a.nfreq; t += blockDim.x) {
    s_wn[t] = a.wn[t];
    s_phi[t] = a.phi[t];
  }
  const int L = xcd_order(a.xcd_remap, blockIdx.x, a.nstep);
  const int tile = L % a.ntile, r = L / a.ntile;
  const bool down = kPairBoth<T> && r >= a.h[0].nrb;
  const int rb = down ? r - a.h[0].nrb : r;
  const HemiArgs<T> h = kPairBoth<T> ? hemi_args(a, down) : a.h[0];
  const HemiArgs<T> hn = kPairBoth<T> ? hemi_pick(A.n[0], A.n[1], down) : A.n[0];
  const int ox = (tile % A.ntx) * kPairX, oy = (tile / A.ntx) * kPairY;
  const int nx = a.nx, ny = a.ny;
  const int ex = min(kPairX, nx - ox), ey = min(kPairY, ny - oy);   // nodes of this tile
  // which group: the same for every lane of a wavefront
  const int grp = __builtin_amdgcn_readfirstlane(threadIdx.x / kPairGroup);
  const int t = threadIdx.x % kPairGroup;
  const int ray = h.ray0 + rb;
  const RayConsts& rc = a.rays[ray];
  const int kO = grp ? hn.kO : h.kO, kM = grp ? hn.kM : h.kM, kP = grp ? hn.kP : h.kP;
  const RayGeom& g1 = layer_geom(a.geom, ray, a.nz, h.kO, h.kM, 0);     // first plane's M
  const RayGeom& g2 = layer_geom(a.geom, ray, a.nz, hn.kO, hn.kM, 0);   // second plane's M
  // the node of this thread: (cx, cy) of its plane's tile
  const int w = grp ? kPairX : kMidX;
  const int cy = t / w, cx = t - cy * w;
  const bool active = grp ? (cx < ex && cy < ey) : (cx <= ex && cy <= ey);
  const bool owner = cx < ex && cy < ey;   // of the rim nodes, the tile they open
  const int fu2 = g2.fu, fv2 = g2.fv;
  const int i = grp ? ox + cx : wrapi(ox + cx + fu2, nx);
  const int j = grp ? oy + cy : wrapi(oy + cy + fv2, ny);
  const int p = active ? j * nx + i : 0;
  PointSetup ps;
  Stencil9 unused;
  setup_point<0>(a.kappa, a.prop, a.emis, a.N, nx, ny, a.np, kO, kM, kP, grp ? g2 : g1,
                 layer_geom(a.geom, ray, a.nz, kO, kP < 0 ? kM : kP, 1), rc, p, a.parabolic != 0,
                 ps, unused);
  T eMv[3], rMv[3], eOv[3], rOv[3];
  kprime_entries(ps.etaM, ps.ikM, eMv, rMv);
  kprime_entries(ps.etaO, ps.ikO, eOv, rOv);
  const auto KO = step_op(eOv, rOv);
  StepSource<T> src[3];
#pragma unroll
  for (int s = 0; s < 3; ++s) step_source(ps.SM[s], ps.SO[s], ps.cM[s], src[s]);
  const T tau0 = (T)ps.tau0M, lf = (T)ps.lamfac;
  const T w00 = (T)ps.sM.w00, w10 = (T)ps.sM.w10, w01 = (T)ps.sM.w01, w11 = (T)ps.sM.w11;

  const size_t fstride = (size_t)a.np * 4;
  const size_t roff = (size_t)rb * a.nfreq * fstride;
  // the upwind node that this thread brings: entry threadIdx.x of the upwind tile
  const T* ip = h.iprev;
  const bool brings = ip && threadIdx.x < kUpX * kUpY;
  if (brings) {
    const int uy = threadIdx.x / kUpX, ux = threadIdx.x - uy * kUpX;
    const int ui = wrapi(ox + ux + fu2 + g1.fu, nx), uj = wrapi(oy + uy + fv2 + g1.fv, ny);
    ip += roff + 4 * ((size_t)uj * nx + ui);
  }
  T* out = grp ? hn.inext : h.inext;
  const bool stores = out && active && (grp || owner);
  if (stores) out += roff + 4 * (size_t)p;
  double jacc0 = 0.0, jacc1 = 0.0, jacc2 = 0.0, jacc3 = 0.0, lacc = 0.0;
  const int nf = a.nfreq;
  T bring[4] = {T(0), T(0), T(0), T(0)};
  if (brings) {
    load4(ip, bring);
    lds.up[0].put(threadIdx.x, bring);
    load4(ip + (size_t)min(1, nf - 1) * fstride, bring);
  }
  __syncthreads();
  for (int s = 0; s <= nf; ++s) {
    if (brings) {
      lds.up[(s + 1) & 1].put(threadIdx.x, bring);
      load4(ip + (size_t)min(s + 2, nf - 1) * fstride, bring);
    }
    const int f = s - grp;   // the frequency of this group's step
    if (active && f >= 0 && f < nf) {
      T v[4][4], IM[4];
      if (grp) {
        const int c = cy * kMidX + cx;
        lds.mid[f & 1].get(c, v[0]);
        lds.mid[f & 1].get(c + 1, v[1]);
        lds.mid[f & 1].get(c + kMidX, v[2]);
        lds.mid[f & 1].get(c + kMidX + 1, v[3]);
      } else {
        const int c = cy * kUpX + cx;
        lds.up[f & 1].get(c, v[0]);
        lds.up[f & 1].get(c + 1, v[1]);
        lds.up[f & 1].get(c + kUpX, v[2]);
        lds.up[f & 1].get(c + kUpX + 1, v[3]);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
        IM[q] = bilinear(w00, w10, w01, w11, v[0][q], v[1][q], v[2][q], v[3][q]);
      if (!grp && !ip) {   // the upwind plane is the boundary
        IM[0] = h.ibound;
        IM[1] = IM[2] = IM[3] = T(0);
      }
      const Coefs<T> cf = coefficients(tau0 * s_phi[f]);
      T KI[4], b[4], x[4];
      kprime_apply(eMv, rMv, IM, KI);
      step_rhs(cf, IM, KI, src, b);
      stokes_solve<1>(KO, step_freq(KO, cf.psiO), b, x, (f & 1) && (grp || h.iprev));
      if (!grp) lds.mid[f & 1].put(cy * kMidX + cx, x);
      if (stores) store4_nt(out + (size_t)f * fstride, x);
      const double W = s_wn[f];
      jacc0 = fma_t(W, (double)x[0], jacc0);
      jacc1 = fma_t(W, (double)x[1], jacc1);
      jacc2 = fma_t(W, (double)x[2], jacc2);
      jacc3 = fma_t(W, (double)x[3], jacc3);
      lacc = fma_t(W, (double)lambda_star(cf, lf), lacc);
    }
    __syncthreads();
  }
  double* jp = grp ? hn.jpart : h.jpart;
  if (jp && active && (grp || owner)) {
    jp += (size_t)rb * 5 * a.np + p;
    jp[0] = jacc0;
    jp[(size_t)a.np] = jacc1;
    jp[2 * (size_t)a.np] = jacc2;
    jp[3 * (size_t)a.np] = jacc3;
    jp[4 * (size_t)a.np] = lacc;
  }
}

}  // namespace porta
