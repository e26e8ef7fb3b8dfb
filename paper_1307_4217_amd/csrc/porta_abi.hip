// porta_abi.hip -- host side of the C ABI declared in include/porta.h:
// argument validation, workspace layout and the launch sequence of each call.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <initializer_list>
#include <mutex>
#include <string>

#include "../../include/porta.h"
#include "porta_adjoint.hpp"
#include "porta_faces.hpp"
#include "porta_host.hpp"
#include "porta_kernels.hpp"
#include "porta_pair.hpp"
#include "porta_unpol.hpp"

// Workspace of porta_fs_sweep_noalloc, one copy on every device the library runs on,
// held until the process ends: kScratchLimit for the sweeps it takes (scratch_need), the
// rest for the tables of their rays' geometry.
constexpr size_t kScratchLimit = size_t(64) << 20;
constexpr size_t kScratchBytes = size_t(72) << 20;
static __device__ __align__(256) char scratch[kScratchBytes];

namespace porta {
namespace host {

thread_local std::string g_last_error;

int fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  std::vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_last_error = buf;
  return code;
}

int check_launch(const char* what) {
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(PORTA_EDEVICE, "%s: %s", what, hipGetErrorString(e));
  return PORTA_OK;
}

int validate_prec(int prec) {
  if (prec != PORTA_F64 && prec != PORTA_F32) return fail(PORTA_EINVAL, "unknown precision %d", prec);
  return PORTA_OK;
}

}  // namespace host
}  // namespace porta

namespace {

using namespace porta;
using namespace porta::host;

constexpr size_t kAlign = 256;
inline size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

// ---------------------------------------------------------------------------
// Validation
// ---------------------------------------------------------------------------
int validate_grid(const porta_grid* g) {
  if (!g) return fail(PORTA_EINVAL, "grid is NULL");
  if (g->nx < 1 || g->ny < 1 || g->nz < 2)
    return fail(PORTA_EINVAL, "grid sizes must be nx >= 1, ny >= 1, nz >= 2 (got %d %d %d)",
                g->nx, g->ny, g->nz);
  const double n = (double)g->nx * g->ny * g->nz;
  if (n * 10.0 >= 9.0e18 || (double)g->nx * g->ny >= 2147483647.0)
    return fail(PORTA_EINVAL, "grid too large");
  if (!(g->lx > 0.0) || !(g->ly > 0.0) || !std::isfinite(g->lx) || !std::isfinite(g->ly))
    return fail(PORTA_EINVAL, "horizontal periods must be positive and finite");
  if (!g->z) return fail(PORTA_EINVAL, "grid z is NULL");
  for (int k = 0; k < g->nz; ++k)
    if (!std::isfinite(g->z[k])) return fail(PORTA_EINVAL, "z[%d] is not finite", k);
  for (int k = 1; k < g->nz; ++k)
    if (!(g->z[k] > g->z[k - 1])) return fail(PORTA_EINVAL, "z must increase strictly (z[%d])", k);
  return PORTA_OK;
}

int validate_quad(const porta_quad* q) {
  if (!q) return fail(PORTA_EINVAL, "quadrature is NULL");
  if (q->nmu < 1 || q->nmu > kMaxMu) return fail(PORTA_EINVAL, "nmu must be in 1..%d", kMaxMu);
  if (q->nchi < 1 || q->nchi > 4096) return fail(PORTA_EINVAL, "nchi must be in 1..4096");
  if (q->nfreq < 1 || q->nfreq > kMaxFreq)
    return fail(PORTA_EINVAL, "nfreq must be in 1..%d", kMaxFreq);
  if (!q->mu || !q->wmu || !q->phi || !q->wfreq)
    return fail(PORTA_EINVAL, "quadrature arrays must not be NULL");
  double sw = 0.0;
  for (int a = 0; a < q->nmu; ++a) {
    if (!(q->mu[a] > 0.0 && q->mu[a] <= 1.0))
      return fail(PORTA_EINVAL, "mu[%d] = %g is not in (0, 1]", a, q->mu[a]);
    if (!(q->wmu[a] >= 0.0) || !std::isfinite(q->wmu[a]))
      return fail(PORTA_EINVAL, "wmu[%d] must be finite and >= 0", a);
    sw += q->wmu[a];
  }
  if (std::fabs(sw - 1.0) > 1e-12) return fail(PORTA_EINVAL, "wmu must sum to 1 (sum = %.17g)", sw);
  double sf = 0.0;
  for (int j = 0; j < q->nfreq; ++j) {
    if (!(q->phi[j] > 0.0) || !std::isfinite(q->phi[j]))
      return fail(PORTA_EINVAL, "phi[%d] must be finite and > 0", j);
    if (!(q->wfreq[j] >= 0.0) || !std::isfinite(q->wfreq[j]))
      return fail(PORTA_EINVAL, "wfreq[%d] must be finite and >= 0", j);
    sf += q->wfreq[j] * q->phi[j];
  }
  if (!(sf > 0.0)) return fail(PORTA_EINVAL, "sum of wfreq * phi must be > 0");
  return PORTA_OK;
}

int validate_interp(int interp) {
  if (interp != PORTA_INTERP_BILINEAR && interp != PORTA_INTERP_BEZIER2D)
    return fail(PORTA_EINVAL, "unknown interpolation mode %d", interp);
  return PORTA_OK;
}

size_t elem(int prec) { return prec == PORTA_F32 ? sizeof(float) : sizeof(double); }

// Tiles per XCD per round of the plane kernels (measured best on MI355X: 8).
int xcd_chunk(const porta_options* o) { return (o && o->xcd_remap >= 0) ? o->xcd_remap : 8; }
int parabolic_of(const porta_options* o) { return (o && o->control == PORTA_CONTROL_PARABOLIC) ? 1 : 0; }
// Stokes parameters carried by the sweep: 4, or 1 for the unpolarized problem.
int nstokes(const porta_options* o) { return (o && o->stokes == 1) ? 1 : 4; }

int validate_options(const porta_options* o) {
  if (!o) return PORTA_OK;
  if (o->ray_batch < 0 || o->block < 0 || o->xcd_remap < -1)
    return fail(PORTA_EINVAL, "ray_batch and block must be >= 0, xcd_remap >= -1");
  if (o->control != PORTA_CONTROL_BESSER && o->control != PORTA_CONTROL_PARABOLIC)
    return fail(PORTA_EINVAL, "unknown control point rule %d", o->control);
  if (o->stokes != 0 && o->stokes != 1 && o->stokes != 4)
    return fail(PORTA_EINVAL, "stokes must be 0 or 4 (Stokes vector) or 1 (intensity only)");
  if (o->ray_count < 0 || o->ray_first < 0)
    return fail(PORTA_EINVAL, "ray_first and ray_count must be >= 0");
  if (o->check_inputs != 0 && o->check_inputs != 1)
    return fail(PORTA_EINVAL, "check_inputs must be 0 or 1");
  if (o->faces != 0 && o->faces != 1) return fail(PORTA_EINVAL, "faces must be 0 or 1");
  if (o->faces_chunk < 0) return fail(PORTA_EINVAL, "faces_chunk must be >= 0");
  return PORTA_OK;
}

bool faces_of(const porta_options* o) { return o && o->faces == 1; }

int validate_rays(const porta_quad* q, const porta_options* o) {
  if (o && o->ray_count > 0 && (int64_t)o->ray_first + o->ray_count > 2LL * q->nmu * q->nchi)
    return fail(PORTA_EINVAL, "ray range %d + %d beyond the %d rays", o->ray_first, o->ray_count,
                2 * q->nmu * q->nchi);
  return PORTA_OK;
}

// Rays of the call: [first, first + count) of the enumeration (upward rays first), all
// rays when count is 0; the part of it in one hemisphere as [lo, hi) of 0..nh-1.
void hemi_range(const porta_quad* q, const porta_options* o, int hemi, int& lo, int& hi) {
  const int nh = q->nmu * q->nchi;
  const int first = (o && o->ray_count > 0) ? o->ray_first : 0;
  const int last = (o && o->ray_count > 0) ? o->ray_first + o->ray_count : 2 * nh;
  lo = std::max(first, hemi * nh) - hemi * nh;
  hi = std::min(last, (hemi + 1) * nh) - hemi * nh;
  if (hi < lo) hi = lo;
}

int hemi_count(const porta_quad* q, const porta_options* o, int hemi) {
  int lo, hi;
  hemi_range(q, o, hemi, lo, hi);
  return hi - lo;
}

// Rays swept together: the options' batch, at most the call's rays in one hemisphere.
int ray_batch(const porta_quad* q, const porta_options* o) {
  const int nh = q->nmu * q->nchi;
  const int rb = (o && o->ray_batch > 0) ? o->ray_batch : nh;
  return std::min(rb, std::max({1, hemi_count(q, o, 0), hemi_count(q, o, 1)}));
}

// ---------------------------------------------------------------------------
// How a plane step is cut into blocks
// ---------------------------------------------------------------------------
constexpr int kCus = 256;

// A launch has fewer than 2^32 threads in each dimension.
bool fits_launch(int64_t blocks, int threads) { return blocks <= 0xffffffffLL / threads; }

// Nodes per block of the plane kernels: the options' choice, else 256, fewer on planes
// that fit in fewer wavefronts.
int plane_block(const porta_grid* g, const porta_options* o) {
  if (o && o->block > 0) return o->block;
  const int64_t np = (int64_t)g->nx * g->ny;
  return np >= 256 ? 256 : (int)((np + 63) / 64 * 64);
}

int64_t plane_tiles(const porta_grid* g, const porta_options* o) {
  const int block = plane_block(g, o);
  return ((int64_t)g->nx * g->ny + block - 1) / block;
}

// Frequency chunks of a launch of `blocks` blocks that would each hold every frequency.
// Every chunk repeats the set-up of its nodes (kSetup updates' worth: 4 to 8 measured from
// the cost of chunks on a full chip), so chunks pay only where CUs stay idle: the count
// minimises (kSetup + frequencies per chunk) x blocks per CU, rounded up.  Time per plane
// step with 1, 2, 3, 4, 6 chunks: FP64 16x16 nodes, 80 rays (80 blocks), 21 frequencies:
// 22.5, 16.5, 15.8, 19.1, 18.3 us; FP32 32x32, 24 rays (96 blocks), 41 frequencies: 25.4,
// 17.3, 19.2, 18.6, 19.5; FP64 32x32, 80 rays (320 blocks): 43.2, 43.0, 45.9, 51.7, 61.1;
// FP64 64x64, 80 rays (1280 blocks): 213, 231, 250, 279, 319.
// least: the part of the time of one chunk, 1/least, that chunks have to save (0: any).
int freq_chunks(int64_t blocks, int nfreq, int64_t least = 0) {
  constexpr int64_t kSetup = 6, kMaxChunks = 32;
  int best = 1;
  int64_t cost = 0, one = 0;
  for (int n = 1; n <= std::min<int64_t>(nfreq, kMaxChunks); ++n) {
    // no n from here on costs less than its share of the chip, without the rounding up
    if (n > 1 && (kSetup * n + nfreq) * blocks >= cost * kCus) break;
    const int64_t per = (nfreq + n - 1) / n;
    if (n > 1 && per == (nfreq + n - 2) / (n - 1)) continue;   // no shorter chunk than n - 1
    const int64_t c = (kSetup + per) * ((blocks * n + kCus - 1) / kCus);
    if (n == 1) one = c;
    if (n == 1 || c < cost) {
      best = n;
      cost = c;
    }
  }
  return least > 0 && (one - cost) * least < one ? 1 : best;
}

// Chunks of the launches of an adjoint, whose partials the gather reads chunk by chunk.  They have
// to save 1/8 unless they stay long and, in FP32 and the 9-point mode, a chunk's blocks have CUs
// to themselves.  Adjoints of 9 planes with chunks by the cost alone and so: bilinear FP32
// 101x71, 4 rays, 3 frequencies 0.281, 0.260 ms; 236x307, 3 rays, 50 frequencies 2.41, 2.14; FP64
// 206x205, 1 ray, 24 frequencies 0.827, 0.751; 9-point FP32 142x156, 4 rays, 17 frequencies 2.11,
// 1.76; 190x263, 2 rays, 111 frequencies 7.23, 6.30; FP64 131x137, 6 rays, 69 frequencies 9.92,
// 9.19.  Those that stay by the cost alone, with chunks and without: bilinear FP64 121x183, 12 rays,
// 113 frequencies 12.2, 12.8; 162x136, 6 rays, 40 frequencies 2.80, 2.94; FP32 48x62, 12 rays, 29
// frequencies 0.43, 0.48; 9-point FP32 60x70, 12 rays, 127 frequencies 5.82, 6.26.
template <class T>
int adjoint_chunks(int64_t blocks, int nfreq, int interp) {
  const bool bil = interp == PORTA_INTERP_BILINEAR;
  const bool any = nfreq >= (bil ? 25 : 80) && (blocks < kCus || (bil && sizeof(T) == 8));
  return freq_chunks(blocks, nfreq, any ? 0 : 8);
}

// The cut of a sweep: whether the two hemispheres' batches share launches, and the
// frequency chunks.  Sharing halves the number of dependent launches and fills each of
// them; it takes the plane states of both batches, so it is for launches that leave
// room on the chip (at most kShareBlocks blocks, about 8 per CU, from one hemisphere) and whose
// states do not fill the memory (kShareBytes, 1/36 of it, for both).
struct SweepPlan {
  int nrb;         // rays of a batch in one hemisphere
  bool share;      // an upward and a downward batch per launch
  bool pair;       // two planes per launch (porta_pair.hpp)
  bool chunks;     // frequency chunks (FP64: their partial sums change the order of the sums
                   // over frequencies that make J, which in an FP32 iteration would tip
                   // the rounding of the next emissivities)
  int rows;        // rays whose states the workspace holds: nrb, or those of both batches
  size_t jrows;    // (ray, chunk) rows of partial sums the workspace holds
  int window;      // layers of the rays' geometry that the workspace holds (0: all, of all rays)
  bool few;        // first faces: the cut with the fewest chunks (faces_shape)
};
constexpr int64_t kShareBlocks = 2048;
constexpr size_t kShareBytes = size_t(8) << 30;

// Sweeps whose planes can go in pairs: bilinear Stokes-vector plane hops at the default block
// size (the 9-point mode, known only at the call, goes plane by plane).
bool pair_of(const porta_options* o) {
  return nstokes(o) == 4 && !faces_of(o) && !(o && o->block > 0);
}

// Whether two planes take less time by a launch of both (pairs of `rows` rays) than by two of
// one (rows in n frequency chunks): a pair reads and writes half the states, but its set-up
// is not spread over as many wavefronts, its tiles have a rim, and its blocks are twice as
// large.  Times in us: rounds of the chip, times the frequencies and a set-up in units of them,
// times the time of one.  Measured (rows of both hemispheres where they share launches), pairs
// and planes, a sweep: FP64 128x128x33, 40 rays, 2, 7, 12 frequencies 6.3 and 4.4, 8.5 and
// 7.6, 10.7 and 10.4 ms; 256x256x17, 41 frequencies 44.1 and 54.0; shared, 64x64x49, 5, 31, 101
// frequencies 2.8 and 2.5, 7.1 and 8.0, 19.3 and 24.1; 37x30x45, 80 rays, 31 frequencies
// (9 tiles for 1110 nodes) 5.5 and 5.0.  FP32 256x256, 40 rays, 9 and 41 frequencies, 33 and 17
// planes 19.3 and 16.2, 21.7 and 22.5; 256x256x128, 101 frequencies 738 and 845.
bool pair_faster(const porta_grid* g, int prec, int64_t tiles, int64_t rows, int nfreq, int n) {
  const bool f64 = prec == PORTA_F64;
  // the tables of the frequencies and the tiles within 64 KiB of LDS
  if (nfreq * (f64 ? 16 : 12) + (f64 ? sizeof(PairLds<double>) : sizeof(PairLds<float>)) > 65536)
    return false;
  const int64_t pairs = pair_tiles(g->nx, g->ny) * rows, slots = f64 ? kCus : 2 * kCus;
  // (below a wavefront per SIMD an update takes about half as long as with two)
  const double rounds = std::max(0.5, double(tiles * rows * n) / (f64 ? 2 * kCus : 3 * kCus));
  const int per = (nfreq + n - 1) / n;
  const double pair = double((pairs + slots - 1) / slots) *
                      (f64 ? 1.02 * (12.5 + nfreq) : 0.96 * (17.0 + nfreq));
  const double plane = 2.0 * rounds * (f64 ? 1.91 * (5.1 + per) : 1.07 * (9.5 + per));
  return pair < plane;
}

// The geometry of every ray on every layer takes 64 bytes each; from kGeomBytes on (160 rays on
// 26 thousand layers, 8192 on 512) a call holds that of one batch on a window of layers, which it
// makes anew as the march moves on.  A window serves one hemisphere, plane by plane.
constexpr size_t kGeomBytes = size_t(256) << 20;
constexpr size_t kGeomEntry = 2 * sizeof(RayGeom);

int geom_window(const porta_grid* g, const porta_quad* q, size_t rays) {
  if (2 * (size_t)q->nmu * q->nchi * (g->nz - 1) * kGeomEntry <= kGeomBytes) return 0;
  const size_t n = std::max<size_t>(2, kGeomBytes / (rays * kGeomEntry));
  return (int)std::min<size_t>(n, g->nz - 1);
}

// Rays of a batch in one hemisphere.
int sweep_batch(const porta_grid* g, const porta_quad* q, const porta_options* o) {
  // a launch is one row of at most 2^31 threads
  const int64_t most = std::max<int64_t>(1, (1 << 23) / plane_tiles(g, o));
  const int nrb = (int)std::min<int64_t>(ray_batch(q, o), most);
  return faces_of(o) ? std::min(nrb, 6553) : nrb;   // 5 blocks per ray in a grid's z of 65535
}

// The largest batch whose launches both hemispheres share.
int share_batch(const porta_grid* g, const porta_quad* q, int prec, const porta_options* o) {
  const size_t state = (size_t)g->nx * g->ny * q->nfreq * nstokes(o) * elem(prec);
  if (!faces_of(o) && geom_window(g, q, 1)) return 0;
  return (int)std::min<size_t>(kShareBlocks / plane_tiles(g, o), kShareBytes / (4 * state));
}

// Whether the reduction of J is launches of its own, kJWideNodes nodes a block (FP64: a group of
// the rays in a wavefront, its constants by scalar loads; FP32, in order: a node a thread): the
// kernels of the plane steps leave it two wavefronts per SIMD, and large planes take several
// rounds of the chip without it.  Sweeps of 9 planes on its own and within the plane steps: FP64,
// 3 frequencies, 4 rays 160x160 0.34, 0.33 ms; 200x200 0.42, 0.48; 256x256 0.58, 0.74; 400x400
// 1.39, 1.94; 40 rays 128x128 1.35, 1.25; 160x160 2.02, 1.98; 200x200 2.96, 3.11; 256x256 4.57,
// 4.99; 10 frequencies 128x240, 4, 8, 16 and 40 rays 0.55, 0.55; 0.90, 1.02; 1.69, 1.82; 4.13, 4.31.
// FP32, 4 frequencies, 2, 4 and 16 rays 200x200 0.25, 0.24; 0.39, 0.31; 1.10, 0.82; 256x256 0.30,
// 0.36; 0.47, 0.46; 1.40, 1.24; 300x300 0.37, 0.47; 0.60, 0.63; 1.87, 1.78; 400x400 0.56, 0.84; 0.97,
// 1.18; 2.96, 3.22; 1000x1024 3.10, 5.99; 5.22, 7.88; 18.1, 21.1; 3 rays 256x256 0.37, 0.41; 6 rays
// 300x300 0.84, 0.86.
constexpr int kJWide = 30720, kJWideNodes = 64;
bool jwide(int prec, int np, int nrb) {
  if (prec == PORTA_F64) return np >= kJWide;
  return np >= (nrb <= 3 ? 65536 : nrb <= 6 ? 81920 : 131072);
}

// The cut for launches of `rows` rays, `nrb` of them in a hemisphere.
SweepPlan plan_rows(const porta_grid* g, const porta_quad* q, int prec, const porta_options* o,
                    int nrb, int rows) {
  SweepPlan P;
  const int64_t tiles = plane_tiles(g, o);
  P.nrb = nrb;
  P.share = rows > nrb;
  P.rows = rows;
  P.chunks = prec == PORTA_F64;
  const int n = P.chunks ? freq_chunks(tiles * rows, q->nfreq) : 1;
  P.jrows = (size_t)rows * n;
  P.window = faces_of(o) ? 0 : geom_window(g, q, nrb);
  P.few = false;
  // (a pair of launches of both hemispheres: kPairBoth)
  const int np = g->nx * g->ny;
  const int64_t jb = jwide(prec, np, nrb) ? 0 : (int64_t)jblocks(np) * (prec == PORTA_F64 ? 4 : 2);
  P.pair = pair_of(o) && P.window == 0 && (prec == PORTA_F64 || tiles * nrb > kShareBlocks) &&
           fits_launch((int64_t)pair_tiles(g->nx, g->ny) * rows + jb, kPairThreads) &&
           pair_faster(g, prec, tiles, rows, q->nfreq, n);
  return P;
}

SweepPlan sweep_plan(const porta_grid* g, const porta_quad* q, int prec, const porta_options* o) {
  const int nrb = sweep_batch(g, q, o), up = hemi_count(q, o, 0), down = hemi_count(q, o, 1);
  const bool share = nrb <= share_batch(g, q, prec, o) && up > 0 && down > 0;
  return plan_rows(g, q, prec, o, nrb, share ? std::min(nrb, up) + std::min(nrb, down) : nrb);
}

// The most frequencies that a first-face sweep takes in options.faces_chunk, and it needs room for
// one: those whose rows fit kFacesLds beside the tables of every frequency.  (A block keeps
// tables of its own chunk only; what the option and the scratch's rule allow does not depend on
// the cut.)
size_t faces_fit(const porta_grid* g, const porta_quad* q, int prec) {
  const int lanes = (std::max(g->nx, g->ny) + 63) / 64 * 64;
  const size_t base = prec == PORTA_F32 ? faces_col_offset<float>(q->nfreq)
                                        : faces_col_offset<double>(q->nfreq);
  const size_t row = (size_t)(lanes + 4 * (lanes / 64)) * 4 * sizeof(double);
  return kFacesLds > base ? (kFacesLds - base) / row : 0;
}

// The cut of the first-face march for a launch of `rays` rays (porta_faces.hpp): columns,
// ways and frequencies of a block.  The options' faces_chunk, if given, is the chunk of one
// way.  few: as many frequencies in turn as a thread takes at most, however few the rays, so
// that the partial sums of the chunks take the least memory.  fchunk is 0 if it does not fit the
// LDS.
struct FacesShape {
  int lanes, ways, fchunk, nchunk;
};

template <class T>
FacesShape faces_shape_t(const porta_grid* g, const porta_quad* q, const porta_options* o,
                         int rays, bool few) {
  FacesShape S;
  const int nf = q->nfreq;
  S.lanes = (std::max(g->nx, g->ny) + 63) / 64 * 64;
  auto fit = [&](int ways, int want) {   // the chunk that fits, `ways` sets of at most want/ways
    while (want > 0 && faces_lds_bytes<T>(want, S.lanes, ways) > kFacesLds) want -= ways;
    return std::max(want, 0);
  };
  S.ways = 1;
  if (o && o->faces_chunk > 0) {
    const int want = std::min(o->faces_chunk, nf);
    S.fchunk = faces_lds_bytes<T>(want, S.lanes, 1) <= kFacesLds ? want : 0;
  } else {
    // frequencies in turn in one thread: one while their wavefronts fit on the chip
    const int64_t waves = (int64_t)rays * nf * (S.lanes / 64);
    const int64_t rounds = (waves + faces_waves<T>() - 1) / faces_waves<T>();
    const int serial = few ? faces_serial<T>() : (int)std::min<int64_t>(faces_serial<T>(), rounds);
    const int ways = std::min({kFacesMaxWays, kFacesThreads / S.lanes, nf});
    if (serial == 1 && ways > 1) {
      S.fchunk = fit(1, ways);   // one frequency per way: as many ways as fit
      while (S.fchunk > 1 && faces_lds_bytes<T>(S.fchunk, S.lanes, S.fchunk) > kFacesLds) --S.fchunk;
    } else {
      S.fchunk = fit(1, std::min(serial, nf));
    }
    if (S.fchunk > 0) {   // even chunks
      const int n = (nf + S.fchunk - 1) / S.fchunk;
      S.fchunk = (nf + n - 1) / n;
      if (serial == 1 && ways > 1) S.ways = S.fchunk;
    }
  }
  S.nchunk = S.fchunk > 0 ? (nf + S.fchunk - 1) / S.fchunk : 1;
  return S;
}

FacesShape faces_shape(const porta_grid* g, const porta_quad* q, int prec, const porta_options* o,
                       int rays, bool few = false) {
  return prec == PORTA_F32 ? faces_shape_t<float>(g, q, o, rays, few)
                           : faces_shape_t<double>(g, q, o, rays, few);
}

// The cut without sharing and chunks, which needs the least workspace (no more than scratch_need
// counts, and the geometry).
SweepPlan least_plan(const porta_grid* g, int nrb) {
  return {nrb, false, false, false, nrb, (size_t)nrb, std::min(2, g->nz - 1), true};
}

// Chunks of a launch of `rays` rays (each chunk has a row of partial sums).
int launch_chunks(const porta_grid* g, const porta_quad* q, const porta_options* o,
                  const SweepPlan& P, int rays) {
  const int n = P.chunks ? freq_chunks(plane_tiles(g, o) * rays, q->nfreq) : 1;
  return (int)std::max<size_t>(1, std::min<size_t>(n, P.jrows / std::max(rays, 1)));
}

// ---------------------------------------------------------------------------
// Workspace layout (every region 256-byte aligned)
// ---------------------------------------------------------------------------
struct Layout {
  size_t stage;     // doubles: mu[nmu], wmu[nmu], phi[nfreq], wfreq[nfreq], z[nz]
  size_t rays;      // RayConsts[nrays]
  size_t geom;      // RayGeom[nrays][nz - 1][2], or of a batch and a window of layers
  int window;       // layers of that window, 0: all
  size_t phiT;      // T[nfreq]
  size_t wn;        // double[nfreq]
  size_t flag;      // int: result of the optional input check
  size_t end_tables;
  size_t stateA, stateB;   // sweep plane states
  size_t jpart;
  // adjoint: checkpoints, recompute slots, Lambda ping-pong, per-ray partials, gradient
  size_t ck, slots, lamA, lamB, go, gm, gp, grad;
  size_t tf;               // first-face sweep: transposed transfer coefficients
  size_t fcache;           // first-face sweep: set-up of the nodes of a plane
  FacesShape fshape;       // first-face sweep: the cut of its march
  size_t plane;            // bytes of one plane state of a ray batch
  int nck, nslot, stride;  // stride: planes from one checkpoint to the next
  size_t total;
};

// nz: planes whose ray geometry the tables hold (0: none); window: layers of it at a time, for
// `batch` rays (0: all of both).
Layout tables_layout(const porta_quad* q, int prec, int nz, int window = 0, int batch = 0) {
  Layout L{};
  const size_t nrays = 2 * (size_t)q->nmu * q->nchi;
  const size_t planes = window > 0 ? window + 1 : nz;
  size_t off = 0;
  L.stage = off;
  off = align_up(off + sizeof(double) * (2 * (size_t)q->nmu + 2 * (size_t)q->nfreq + planes));
  L.rays = off;
  off = align_up(off + sizeof(RayConsts) * nrays);
  L.geom = off;
  L.window = window;
  if (planes > 0) off = align_up(off + kGeomEntry * (window > 0 ? batch : nrays) * (planes - 1));
  L.phiT = off;
  off = align_up(off + elem(prec) * q->nfreq);
  L.wn = off;
  off = align_up(off + sizeof(double) * q->nfreq);
  L.flag = off;
  off = align_up(off + sizeof(int));
  L.end_tables = off;
  L.total = off;
  return L;
}

Layout sweep_layout(const porta_grid* g, const porta_quad* q, int prec, const porta_options* o,
                    const SweepPlan& P) {
  // (the first-face kernels form their own geometry)
  Layout L = faces_of(o) ? tables_layout(q, prec, 0)
                         : tables_layout(q, prec, g->nz, P.window, P.nrb);
  const size_t np = (size_t)g->nx * g->ny;
  const size_t state = (size_t)P.rows * q->nfreq * np * nstokes(o) * elem(prec);
  size_t off = L.end_tables;
  L.stateA = off;
  off = align_up(off + state);
  L.stateB = off;
  off = align_up(off + state);
  L.jpart = off;
  // double-buffered partial sums, of one plane or two
  off = align_up(off + (P.pair ? 4 : 2) * P.jrows * (nstokes(o) + 1) * np * sizeof(double));
  if (faces_of(o)) {
    // per-chunk partial sums of the first-face kernel
    L.fshape = faces_shape(g, q, prec, o, P.rows, P.few);
    L.ck = off;
    off = align_up(off + (size_t)P.rows * L.fshape.nchunk * 5 * np * sizeof(double));
    // the transfer coefficients with x and y exchanged in every plane
    L.tf = off;
    off = align_up(off + 13 * np * g->nz * elem(prec));
    // the set-up of every node and ray of one plane
    L.fcache = off;
    off = align_up(off + (size_t)P.rows * kFacesCache * np * elem(prec));
  }
  L.total = off;
  return L;
}

// Bytes that serve a sweep with these options and any of fewer rays, a part of the range or a
// smaller batch: those may be cut otherwise (both hemispheres in a launch, more chunks, two
// planes) and take more than a larger one.
size_t sweep_bytes(const porta_grid* g, const porta_quad* q, int prec, const porta_options* o) {
  const int nrb = sweep_batch(g, q, o);
  const int rows = std::max(nrb, 2 * std::min(nrb, share_batch(g, q, prec, o)));
  size_t n = 0;
  for (int r = 1; r <= rows; ++r) {
    const SweepPlan P = plan_rows(g, q, prec, o, std::min(r, nrb), r);
    n = std::max(n, sweep_layout(g, q, prec, o, P).total);
  }
  return n;
}

// Forward states of a batch of rays that the adjoint keeps without being asked (1/288 of
// the device memory): recomputing planes from checkpoints saves nothing worth having below.
constexpr size_t kKeepAllBytes = size_t(1) << 30;

// Checkpoint planes are k = C, 2C, ... <= nz - 2 (the top plane is recomputed).
int checkpoint_count(int nz, int C) { return nz >= 3 ? (nz - 2) / C : 0; }
bool is_checkpoint(int k, int nz, int C) { return k >= 1 && k % C == 0 && k <= nz - 2; }

// What decides whether porta_fs_sweep_noalloc takes a sweep: the plane states and partial
// sums of one hemisphere's batch with every frequency in one chunk (first faces: chunks of at
// most 4 frequencies in FP32 and 7 in FP64), the ray tables and the first-face set-up.
size_t scratch_need(const porta_grid* g, const porta_quad* q, int prec, const porta_options* o) {
  const size_t np = (size_t)g->nx * g->ny, nf = q->nfreq, e = elem(prec);
  const size_t nrb = (size_t)ray_batch(q, o);
  size_t n = align_up(sizeof(double) * (2 * kMaxMu + 2 * nf)) +
             align_up(sizeof(RayConsts) * 2 * q->nmu * q->nchi) + align_up(e * nf) +
             align_up(sizeof(double) * nf) + align_up(sizeof(int));
  n += 2 * align_up(nrb * nf * np * nstokes(o) * e) + align_up(2 * nrb * 5 * np * sizeof(double));
  if (faces_of(o)) {
    size_t chunk = std::min<size_t>({prec == PORTA_F32 ? 4u : 7u, faces_fit(g, q, prec), nf});
    if (o->faces_chunk > 0) chunk = std::min<size_t>(o->faces_chunk, nf);
    chunk = std::max<size_t>(chunk, 1);
    const size_t nchunk = (nf + chunk - 1) / chunk;
    n += align_up(nrb * nchunk * 5 * np * sizeof(double)) + align_up(13 * np * g->nz * e) +
         align_up(nrb * 26 * np * e);
  }
  return n;
}

// Adjoint: checkpoint planes (unless the caller brings them), C slots for the
// planes recomputed between two checkpoints, two planes of Lambda, the
// per-(node, ray) partials of one plane and the FP64 gradient accumulator.
Layout adjoint_layout(const porta_grid* g, const porta_quad* q, int prec, int stride,
                      const porta_options* o, bool own_checkpoints, size_t nrb) {
  Layout L = tables_layout(q, prec, g->nz, geom_window(g, q, nrb), (int)nrb);
  const size_t np = (size_t)g->nx * g->ny, N = np * g->nz;
  L.plane = nrb * q->nfreq * np * 4 * elem(prec);
  // planes of its own that are small enough are all kept, whatever the stride
  L.stride = own_checkpoints && L.plane * g->nz <= kKeepAllBytes ? 1 : stride;
  L.nck = own_checkpoints ? checkpoint_count(g->nz, L.stride) : 0;
  L.nslot = L.stride;
  // rows of partials: one for each ray and frequency chunk
  const size_t nrow = nrb * freq_chunks(plane_tiles(g, o) * nrb, q->nfreq);
  size_t off = L.end_tables;
  L.ck = off;
  off = align_up(off + (size_t)L.nck * L.plane);
  L.slots = off;
  off = align_up(off + (size_t)L.nslot * L.plane);
  L.lamA = off;
  off = align_up(off + L.plane);
  L.lamB = off;
  off = align_up(off + L.plane);
  // per-(node, ray) partials in the sweep precision
  L.go = off;
  off = align_up(off + nrow * 13 * np * elem(prec));
  L.gm = off;
  off = align_up(off + nrow * 13 * np * elem(prec));
  L.gp = off;
  off = align_up(off + nrow * 7 * np * elem(prec));
  L.grad = off;
  off = align_up(off + 13 * N * sizeof(double));
  L.total = off;
  return L;
}

// Bytes that serve an adjoint with these options and any of fewer rays: a smaller batch may keep
// every plane or be cut into more chunks.
size_t adjoint_bytes(const porta_grid* g, const porta_quad* q, int prec, int stride,
                     const porta_options* o, bool own_checkpoints) {
  size_t n = 0;
  for (int r = ray_batch(q, o); r >= 1; --r)
    n = std::max(n, adjoint_layout(g, q, prec, stride, o, own_checkpoints, r).total);
  return n;
}

// Checkpoints hold the upward rays of the call's ray range:
// [(nz-2)/C][upward rays of the range][nfreq][ny][nx][4].
size_t checkpoint_bytes(const porta_grid* g, const porta_quad* q, int prec, int stride,
                        const porta_options* o) {
  int lo, hi;
  hemi_range(q, o, 0, lo, hi);
  return (size_t)checkpoint_count(g->nz, stride) * (hi - lo) * q->nfreq *
         ((size_t)g->nx * g->ny) * 4 * elem(prec);
}

// Upload host doubles through kernel arguments (ordered on the stream), one array after
// the other; as few launches as the argument block allows.
struct HostArray {
  const double* p;
  size_t n;
};

int upload(double* dst, std::initializer_list<HostArray> arrays, hipStream_t st) {
  UploadChunk c;
  c.dst = dst;
  c.n = 0;
  auto flush = [&]() {
    hipLaunchKernelGGL(k_upload, dim3(1), dim3(256), 0, st, c);
    c.dst += c.n;
    c.n = 0;
  };
  for (const HostArray& a : arrays)
    for (size_t o = 0; o < a.n;) {
      const size_t m = std::min<size_t>(kUploadChunk - c.n, a.n - o);
      std::memcpy(c.v + c.n, a.p + o, sizeof(double) * m);
      c.n += (int)m;
      o += m;
      if (c.n == kUploadChunk) flush();
    }
  if (c.n) flush();
  return check_launch("upload");
}

// The geometry of the rays: the table of a call (k_prepare), or a window of it.
struct Geometry {
  const porta_grid* g;
  const porta_quad* q;
  GeomArgs a;
  const double* mu;   // device
  int window;         // layers, 0: the table holds everything
  int l0;             // first layer of the window

  // The layers next to plane k for these rays, before a launch that solves it (dir: the way the
  // planes go).  Makes a window that starts, or for dir < 0 ends, with them unless they are there.
  int need(int ray0, int nray, int k, int dir, hipStream_t st) {
    const int lo = std::max(k - 1, 0), hi = std::min(k + 1, g->nz - 1);
    if (window == 0 || (ray0 == a.ray0 && nray == a.nray && lo >= l0 && hi <= l0 + a.nl))
      return PORTA_OK;
    l0 = dir > 0 ? lo : std::max(0, hi - window);
    a.nl = std::min(window, g->nz - 1 - l0);
    a.ray0 = ray0;
    a.nray = nray;
    const int rc = upload(const_cast<double*>(a.z), {{g->z + l0, (size_t)a.nl + 1}}, st);
    if (rc) return rc;
    const size_t nb = ((size_t)nray * a.nl + 255) / 256;
    hipLaunchKernelGGL(k_geom, dim3((unsigned)nb), dim3(256), 0, st, a, mu, q->nmu * q->nchi,
                       q->nchi);
    return check_launch("geom");
  }

  // Where layer_geom finds them.
  template <class Args>
  void set(Args& args) const {
    const ptrdiff_t skip = window ? (ptrdiff_t)a.ray0 * window + l0 : 0;
    args.geom = a.geom - 2 * skip;
    args.nz = a.stride + 1;
  }
};

// The tables of a call; with a grid also the rays' geometry on its layers, as `interp`
// splits it, into `geo`.
template <class T>
int prepare_tables(char* ws, const Layout& L, const porta_grid* g, const porta_quad* q, double w2,
                   int interp, Geometry* geo, hipStream_t st) {
  double* mu = reinterpret_cast<double*>(ws + L.stage);
  double *wmu = mu + q->nmu, *phi = wmu + q->nmu, *wfreq = phi + q->nfreq, *z = wfreq + q->nfreq;
  const int nz = geo && L.window == 0 ? g->nz : 0;   // planes whose layers k_prepare takes
  int rc;
  if ((rc = upload(mu, {{q->mu, (size_t)q->nmu}, {q->wmu, (size_t)q->nmu},
                        {q->phi, (size_t)q->nfreq}, {q->wfreq, (size_t)q->nfreq},
                        {g ? g->z : nullptr, (size_t)nz}}, st)))
    return rc;
  GeomArgs ga{};
  size_t nb = 1;
  if (geo) {
    const int nrays = 2 * q->nmu * q->nchi;
    ga = {z, 0, nz ? nrays : 0, nz ? nz - 1 : 0, nz ? nz - 1 : L.window, g->nx, g->ny,
          g->nx / g->lx, g->ny / g->ly, interp == PORTA_INTERP_BEZIER2D ? 0.5 : 0.0,
          reinterpret_cast<RayGeom*>(ws + L.geom)};
    nb += ((size_t)ga.nray * ga.nl + 255) / 256;
    *geo = {g, q, ga, mu, L.window, 0};
  }
  hipLaunchKernelGGL(k_prepare<T>, dim3((unsigned)nb), dim3(256), 0, st, mu, wmu, q->nmu, q->nchi,
                     w2, phi, wfreq, q->nfreq, reinterpret_cast<RayConsts*>(ws + L.rays),
                     reinterpret_cast<T*>(ws + L.phiT), reinterpret_cast<double*>(ws + L.wn), ga);
  return check_launch("prepare");
}

int fill(double* p, size_t n, double v, hipStream_t st) {
  if (n == 0) return PORTA_OK;
  const size_t blocks = std::min<size_t>((n + 255) / 256, 65536);
  hipLaunchKernelGGL(k_fill_f64, dim3((unsigned)blocks), dim3(256), 0, st, p, n, v);
  return check_launch("fill");
}

// The opt-in input check: one pass over the fields, then a wait on the stream for
// its verdict.
template <class T>
int check_inputs(const porta_grid* g, const porta_fields* f, char* ws, const Layout& L,
                 hipStream_t st) {
  const size_t N = (size_t)g->nx * g->ny * g->nz;
  int* flag = reinterpret_cast<int*>(ws + L.flag);
  hipLaunchKernelGGL(k_zero_flag, dim3(1), dim3(64), 0, st, flag);
  int rc;
  if ((rc = check_launch("zero_flag"))) return rc;
  const size_t blocks = std::min<size_t>((N + 255) / 256, 65536);
  hipLaunchKernelGGL(k_check_fields<T>, dim3((unsigned)blocks), dim3(256), 0, st,
                     static_cast<const T*>(f->kappa), static_cast<const T*>(f->propmat),
                     static_cast<const T*>(f->emis), N, flag);
  if ((rc = check_launch("check_fields"))) return rc;
  int h = 0;
  if (hipMemcpyAsync(&h, flag, sizeof(int), hipMemcpyDeviceToHost, st) != hipSuccess ||
      hipStreamSynchronize(st) != hipSuccess)
    return fail(PORTA_EDEVICE, "reading the input check failed");
  if (h) return fail(PORTA_ENONFINITE, "a transfer coefficient is not finite, or eta_I <= 0");
  return PORTA_OK;
}

template <class T>
int launch_jreduce(double* jkq, const double* jpart, const RayConsts* rays, int ray0, int nrb,
                   int nchunk, int ns, int np, size_t N, size_t plane_off, double ibound,
                   hipStream_t st) {
  const JJob J = {jpart, rays + ray0, nrb, nchunk, ibound, plane_off};
  auto go = [&](auto* kernel, int nodes, int threads) {
    constexpr int most = int(0xffffffffLL / 256);   // fits_launch
    for (int first = 0, all = jblocks(np, nodes); first < all; first += most)
      hipLaunchKernelGGL(kernel, dim3(std::min(all - first, most)), dim3(threads),
                         jlds_bytes(threads, sizeof(T)), st, J, jkq, np, N, first);
  };
  if (jwide(sizeof(T) == 8 ? PORTA_F64 : PORTA_F32, np, nrb)) {
    const int threads = sizeof(T) == 8 ? 256 : kJWideNodes;
    if (ns == 1) go(k_jreduce<1, T, kJWideNodes>, kJWideNodes, threads);
    else go(k_jreduce<4, T, kJWideNodes>, kJWideNodes, threads);
  } else {
    if (ns == 1) go(k_jreduce<1, T, kJNodes>, kJNodes, 256);
    else go(k_jreduce<4, T, kJNodes>, kJNodes, 256);
  }
  return check_launch("jreduce");
}

// The batches of a sweep in turn: walk(r0, nr) with the first ray and the number of rays of
// either hemisphere, together where the plan shares launches.  up_only: nothing that the
// call returns depends on the downward rays (no J).
template <class Walk>
int walk_batches(const porta_quad* q, const porta_options* o, const SweepPlan& P, bool up_only,
                 Walk walk) {
  int rc, lo[2], hi[2];
  for (int m = 0; m < 2; ++m) hemi_range(q, o, m, lo[m], hi[m]);
  if (up_only) hi[1] = lo[1];
  if (P.share) {
    for (int b = 0;; ++b) {
      int r0[2], nr[2];
      for (int m = 0; m < 2; ++m) {
        r0[m] = std::min(lo[m] + b * P.nrb, hi[m]);
        nr[m] = std::min(P.nrb, hi[m] - r0[m]);
      }
      if (nr[0] + nr[1] == 0) return PORTA_OK;
      if ((rc = walk(r0, nr))) return rc;
    }
  }
  for (int m = 0; m < 2; ++m)
    for (int r = lo[m]; r < hi[m]; r += P.nrb) {
      const int n = std::min(P.nrb, hi[m] - r);
      const int r0[2] = {m == 0 ? r : 0, m == 0 ? 0 : r}, nr[2] = {m == 0 ? n : 0, m == 0 ? 0 : n};
      if ((rc = walk(r0, nr))) return rc;
    }
  return PORTA_OK;
}

// ---------------------------------------------------------------------------
// Forward sweep with M and P on the first face crossed (options.faces = 1)
// ---------------------------------------------------------------------------
template <class T>
int sweep_faces_impl(const porta_grid* g, const porta_quad* q, const porta_fields* f,
                     const porta_options* o, double* jkq, T* itop, char* ws, const SweepPlan& P,
                     const Layout& L, hipStream_t st) {
  int rc;
  const int nx = g->nx, ny = g->ny, nz = g->nz, np = nx * ny;
  const size_t N = (size_t)np * nz;
  const int nh = q->nmu * q->nchi;
  const FacesShape& S = L.fshape;
  const RayConsts* rays = reinterpret_cast<const RayConsts*>(ws + L.rays);
  T* state[2] = {reinterpret_cast<T*>(ws + L.stateA), reinterpret_cast<T*>(ws + L.stateB)};
  double* jpart = reinterpret_cast<double*>(ws + L.jpart);
  double* jchunk = reinterpret_cast<double*>(ws + L.ck);
  // rays that meet an x face first read the fields with x and y exchanged
  T* tf = reinterpret_cast<T*>(ws + L.tf);
  {
    const T* src[3] = {static_cast<const T*>(f->kappa), static_cast<const T*>(f->propmat),
                       static_cast<const T*>(f->emis)};
    const size_t nfield[3] = {1, 6, 6}, dst[3] = {0, N, 7 * N};
    for (int c = 0; c < 3; ++c) {
      const size_t n = nfield[c] * N;
      hipLaunchKernelGGL(k_transpose_planes<T>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0,
                         st, src[c], tf + dst[c], nx, ny, nfield[c] * nz);
      if ((rc = check_launch("transpose_planes"))) return rc;
    }
  }
  FacesArgs<T> a{};
  a.kappa = static_cast<const T*>(f->kappa);
  a.prop = static_cast<const T*>(f->propmat);
  a.emis = static_cast<const T*>(f->emis);
  a.kappa_t = tf;
  a.prop_t = tf + N;
  a.emis_t = tf + 7 * N;
  a.rays = rays;
  a.phi = reinterpret_cast<const T*>(ws + L.phiT);
  a.wn = reinterpret_cast<const double*>(ws + L.wn);
  a.jchunk = jkq ? jchunk : nullptr;
  a.cache = reinterpret_cast<T*>(ws + L.fcache);
  a.N = N;
  a.nx = nx;
  a.ny = ny;
  a.np = np;
  a.nfreq = q->nfreq;
  a.fchunk = S.fchunk;
  a.nchunk = S.nchunk;
  a.lanes = S.lanes;
  a.inv_dx = nx / g->lx;
  a.inv_dy = ny / g->ly;
  a.parabolic = parabolic_of(o);
  a.tol = sizeof(T) == 4 ? 0x1p-24 : 0x1p-53;   // the unit roundoff of the sweep precision
  const size_t lds = faces_lds_bytes<T>(S.fchunk, S.lanes, S.ways);
  const bool one = S.ways == S.fchunk;
  const T ibound[2] = {(T)f->i_bottom, T(0)};
  auto walk = [&](const int r0[2], const int nr[2]) -> int {
    const int rows = nr[0] + nr[1];
    const T* prev[2] = {nullptr, nullptr};
    const size_t soff[2] = {0, (size_t)nr[0] * q->nfreq * np * 4};
    const size_t joff[2] = {0, (size_t)nr[0] * 5 * np};
    int e;
    for (int m = 0; m < 2 && jkq; ++m)   // the boundary planes
      if (nr[m] > 0 && (e = launch_jreduce<T>(jkq, nullptr, rays, m * nh + r0[m], nr[m], 1, 4, np, N,
                                           (size_t)(m == 0 ? 0 : nz - 1) * np, (double)ibound[m],
                                           st)))
        return e;
    for (int step = 1; step < nz; ++step) {
      const bool last = (step == nz - 1);
      for (int m = 0; m < 2; ++m) {
        FacesHemi<T>& h = a.h[m];
        const int s = m == 0 ? 1 : -1, k = (m == 0 ? 0 : nz - 1) + s * step;
        h.iprev = prev[m];
        h.top = m == 0 && last && itop;
        h.inext = h.top ? itop + (size_t)r0[m] * q->nfreq * np * 4 : state[step & 1] + soff[m];
        h.kO = k;
        h.kM = k - s;
        h.kP = last ? -1 : k + s;
        h.dzM = std::fabs(g->z[k] - g->z[k - s]);
        h.dzP = last ? 0.0 : std::fabs(g->z[k + s] - g->z[k]);
        h.ray0 = m * nh + r0[m];
        h.nrb = nr[m];
        h.ibound = ibound[m];
        prev[m] = h.inext;
      }
      a.nrb = rows;
      hipLaunchKernelGGL(k_faces_setup<T>, dim3((np + 255) / 256, rows), dim3(256), 0, st, a);
      if ((e = check_launch("faces_setup"))) return e;
      const dim3 grid(faces_grid(rows, S.nchunk)), blk(S.lanes * S.ways);
      if (one)
        hipLaunchKernelGGL((k_sweep_plane_faces<T, true>), grid, blk, lds, st, a);
      else
        hipLaunchKernelGGL((k_sweep_plane_faces<T, false>), grid, blk, lds, st, a);
      if ((e = check_launch("sweep_plane_faces"))) return e;
      if (jkq) {
        const unsigned tiles = (unsigned)((std::max(nx, ny) + kSumTile - 1) / kSumTile);
        hipLaunchKernelGGL(k_sum_chunks, dim3(tiles, tiles, rows * 5), dim3(256), 0, st, jpart,
                           (const double*)jchunk, rays, a.h[0].ray0, nr[0], a.h[1].ray0, S.nchunk,
                           nx, ny, a.inv_dx, a.inv_dy);
        if ((e = check_launch("sum_chunks"))) return e;
        for (int m = 0; m < 2; ++m)
          if (nr[m] > 0 && (e = launch_jreduce<T>(jkq, jpart + joff[m], rays, a.h[m].ray0, nr[m], 1, 4,
                                               np, N, (size_t)a.h[m].kO * np, 0.0, st)))
            return e;
      }
    }
    return PORTA_OK;
  };
  return walk_batches(q, o, P, jkq == nullptr, walk);
}

// ---------------------------------------------------------------------------
// Forward sweep
// ---------------------------------------------------------------------------
// The parts of a plane step's arguments that do not change from plane to plane.
template <class T>
PlaneArgs<T> plane_args(const porta_grid* g, const porta_quad* q, const porta_fields* f,
                        const porta_options* o, char* ws, const Layout& L, const Geometry& geo) {
  PlaneArgs<T> a{};
  a.kappa = static_cast<const T*>(f->kappa);
  a.prop = static_cast<const T*>(f->propmat);
  a.emis = static_cast<const T*>(f->emis);
  a.rays = reinterpret_cast<const RayConsts*>(ws + L.rays);
  geo.set(a);
  a.phi = reinterpret_cast<const T*>(ws + L.phiT);
  a.wn = reinterpret_cast<const double*>(ws + L.wn);
  a.nx = g->nx;
  a.ny = g->ny;
  a.np = g->nx * g->ny;
  a.N = (size_t)a.np * g->nz;
  a.nfreq = q->nfreq;
  a.ntile = (int)plane_tiles(g, o);
  a.xcd_remap = xcd_chunk(o);
  a.parabolic = parabolic_of(o);
  return a;
}

// Planes of O, M and P of a hemisphere's rays on their plane k (s = +-1 along the ray).
template <class T>
void set_plane(HemiArgs<T>& h, const porta_grid* g, int k, int s) {
  const bool last = k + s < 0 || k + s >= g->nz;
  h.kO = k;
  h.kM = k - s;
  h.kP = last ? -1 : k + s;
}

// In FP32 chunks of an even number of frequencies: there the solve rounds c.r by the parity of
// a frequency's place in its chunk (stokes_solve), which is then that of the frequency, and
// the planes that the adjoint sweeps again are those of the sweep bit for bit.
template <class T>
void set_chunks(PlaneArgs<T>& a, int nchunk, int rays) {
  a.fchunk = (a.nfreq + nchunk - 1) / nchunk;
  if (sizeof(T) == 4 && nchunk > 1) a.fchunk += a.fchunk & 1;
  a.nchunk = (a.nfreq + a.fchunk - 1) / a.fchunk;
  a.nstep = a.ntile * rays * a.nchunk;
}

template <class T>
int launch_plane(const PlaneArgs<T>& a, int ns, int interp, int block, hipStream_t st) {
  const size_t tab = (size_t)a.fchunk * (sizeof(double) + sizeof(T));
  const size_t lds = a.njb ? std::max(tab, jlds_bytes(block, sizeof(T))) : tab;
  const dim3 grid(a.nstep + a.njb);
  if (ns == 1)
    hipLaunchKernelGGL(k_sweep_plane_i<T>, grid, dim3(block), lds, st, a);
  else if (interp == PORTA_INTERP_BEZIER2D)
    hipLaunchKernelGGL((k_sweep_plane<T, 1>), grid, dim3(block), lds, st, a);
  else
    hipLaunchKernelGGL((k_sweep_plane<T, 0>), grid, dim3(block), lds, st, a);
  return check_launch("sweep_plane");
}

template <class T>
int sweep_impl(const porta_grid* g, const porta_quad* q, const porta_fields* f, int interp,
               const porta_options* o, double* jkq, int accumulate, T* itop, T* ckpt, int C,
               char* ws, const SweepPlan& P, const Layout& L, hipStream_t st) {
  int rc;
  Geometry geo;
  if ((rc = prepare_tables<T>(ws, L, g, q, f->w2, interp, faces_of(o) ? nullptr : &geo, st)))
    return rc;
  const int nz = g->nz, np = g->nx * g->ny;
  const size_t N = (size_t)np * nz;
  if (jkq && !accumulate)
    if ((rc = fill(jkq, 10 * N, 0.0, st))) return rc;
  const int nh = q->nmu * q->nchi;
  const int ns = nstokes(o);
  const int block = plane_block(g, o);
  if (block % 64 != 0 || block > 256) return fail(PORTA_EINVAL, "block must be 64, 128, 192 or 256");
  const RayConsts* rays = reinterpret_cast<const RayConsts*>(ws + L.rays);
  T* state[2] = {reinterpret_cast<T*>(ws + L.stateA), reinterpret_cast<T*>(ws + L.stateB)};
  if (faces_of(o))
    return sweep_faces_impl<T>(g, q, f, o, jkq, itop, ws, P, L, st);
  double* const jbase = reinterpret_cast<double*>(ws + L.jpart);
  auto wide = [&](const int nr[2]) {
    return jwide(sizeof(T) == 8 ? PORTA_F64 : PORTA_F32, np, std::max(nr[0], nr[1]));
  };
  const size_t jslot = P.jrows * (ns + 1) * np;   // partial sums of one plane
  int up_lo, up_hi;
  hemi_range(q, o, 0, up_lo, up_hi);
  const T ibound[2] = {(T)f->i_bottom, T(0)};
  // where the state of plane k of a batch goes if it is to be kept: I_top, a checkpoint for
  // the adjoint, or nowhere
  auto kept = [&](int m, int k, int r0) -> T* {
    if (m != 0) return nullptr;
    if (k == nz - 1) return itop ? itop + (size_t)r0 * q->nfreq * np * ns : nullptr;
    if (!ckpt || !is_checkpoint(k, nz, C)) return nullptr;
    return ckpt + ((size_t)(k / C - 1) * (up_hi - up_lo) + (r0 - up_lo)) * q->nfreq * np * 4;
  };
  // one launch per plane step for a batch of upward rays, of downward rays, or of both
  auto walk = [&](const int r0[2], const int nr[2]) -> int {
    PlaneArgs<T> a = plane_args<T>(g, q, f, o, ws, L, geo);
    a.jkq = jkq;
    set_chunks(a, launch_chunks(g, q, o, P, nr[0] + nr[1]), nr[0] + nr[1]);
    // states and partial sums of the downward rays follow those of the upward ones
    const size_t soff[2] = {0, (size_t)nr[0] * q->nfreq * np * ns};
    const size_t joff[2] = {0, (size_t)nr[0] * a.nchunk * (ns + 1) * np};
    // the reduction of J rides on the plane steps where it pays
    const bool fused =
        jkq && !wide(nr) && fits_launch((int64_t)a.nstep + 2 * jblocks(np), block);
    a.njb = fused ? 2 * jblocks(np) : 0;
    auto reduce = [&](int m, const double* part, int k) -> int {
      if (nr[m] == 0) return PORTA_OK;
      return launch_jreduce<T>(jkq, part, rays, m * nh + r0[m], nr[m], a.nchunk, ns, np, N,
                               (size_t)k * np, (double)ibound[m], st);
    };
    int e;
    for (int m = 0; m < 2 && jkq && !fused; ++m)
      if ((e = reduce(m, nullptr, m == 0 ? 0 : nz - 1))) return e;
    const T* prev[2] = {nullptr, nullptr};
    for (int step = 1; step < nz; ++step) {
      for (int m = 0; m < 2; ++m) {
        HemiArgs<T>& h = a.h[m];
        const int s = m == 0 ? 1 : -1, k = (m == 0 ? 0 : nz - 1) + s * step;
        set_plane(h, g, k, s);
        h.ray0 = m * nh + r0[m];
        h.nrb = nr[m];
        h.ibound = ibound[m];
        h.iprev = prev[m];
        h.inext = kept(m, k, r0[m]);
        if (!h.inext) h.inext = state[step & 1] + soff[m];
        // plane k writes partial sums into slot step & 1 while the last blocks add
        // those of plane k - s (or the boundary plane) to J
        h.jpart = jkq ? jbase + (step & 1) * jslot + joff[m] : nullptr;
        h.jpart_prev = (jkq && step > 1) ? jbase + ((step - 1) & 1) * jslot + joff[m] : nullptr;
        h.prev_off = (size_t)(k - s) * np;
        prev[m] = h.inext;
        if (nr[m] > 0 && (e = geo.need(h.ray0, nr[m], k, s, st))) return e;
      }
      geo.set(a);
      a.jsame = nr[0] > 0 && nr[1] > 0 && a.h[0].kM == a.h[1].kM;
      if ((e = launch_plane<T>(a, ns, interp, block, st))) return e;
      for (int m = 0; m < 2 && jkq; ++m)   // fused: the last plane of each hemisphere
        if (!fused || step == nz - 1)
          if ((e = reduce(m, a.h[m].jpart, a.h[m].kO))) return e;
    }
    return PORTA_OK;
  };
  // two planes per launch; of an even number of planes the first one goes alone
  auto walk_pairs = [&](const int r0[2], const int nr[2]) -> int {
    PairArgs<T> A{};
    PlaneArgs<T>& a = A.a;
    a = plane_args<T>(g, q, f, o, ws, L, geo);
    a.jkq = jkq;
    const size_t soff[2] = {0, (size_t)nr[0] * q->nfreq * np * ns};
    const size_t joff[2] = {0, (size_t)nr[0] * (ns + 1) * np};
    const int kb[2] = {0, nz - 1}, up[2] = {1, -1};   // boundary planes, directions
    // where the launch's arguments of a hemisphere are; the hemispheres that it has
    const int at[2] = {0, kPairBoth<T> ? 1 : 0}, m0 = nr[0] > 0 ? 0 : 1, m1 = nr[1] > 0 ? 2 : 1;
    auto set = [&](HemiArgs<T>& h, int m, int k, const T* prev, T* next, int slot) {
      set_plane(h, g, k, up[m]);
      h.ray0 = m * nh + r0[m];
      h.nrb = nr[m];
      h.ibound = ibound[m];
      h.iprev = prev;
      h.inext = next;
      h.jpart = jkq ? jbase + slot * jslot + joff[m] : nullptr;
    };
    // planes whose partial sums are still to be added to J
    for (int m = m0; m < m1; ++m) {
      A.jp[at[m]][0] = {nullptr, (size_t)kb[m] * np};
      A.njprev[at[m]] = 1;
    }
    const bool fused = jkq && !wide(nr);
    auto reduce = [&]() -> int {
      for (int m = m0; m < m1; ++m)
        for (int c = 0; c < A.njprev[at[m]]; ++c) {
          const JPrev& j = A.jp[at[m]][c];
          const int rc = launch_jreduce<T>(jkq, j.part, rays, m * nh + r0[m], nr[m], 1, ns, np, N,
                                           j.off, (double)ibound[m], st);
          if (rc) return rc;
        }
      return PORTA_OK;
    };
    const T* prev[2] = {nullptr, nullptr};
    int step = 1, launch = 0, e;
    if (jkq && !fused && (e = reduce())) return e;
    if (nz % 2 == 0) {
      for (int m = m0; m < m1; ++m) {
        const int k = kb[m] + up[m];
        T* next = kept(m, k, r0[m]);
        if (!next) next = state[0] + soff[m];
        set(a.h[at[m]], m, k, nullptr, next, 0);
        a.h[at[m]].prev_off = (size_t)kb[m] * np;
        A.jp[at[m]][0] = {a.h[at[m]].jpart, (size_t)k * np};
        prev[m] = next;
      }
      set_chunks(a, 1, nr[0] + nr[1]);
      a.njb = fused ? 2 * jblocks(np) : 0;
      if ((e = launch_plane<T>(a, ns, interp, block, st))) return e;
      if (jkq && !fused && (e = reduce())) return e;
      step = 2;
      launch = 1;
    }
    A.ntx = (g->nx + kPairX - 1) / kPairX;
    a.ntile = pair_tiles(g->nx, g->ny);
    a.nstep = a.ntile * (nr[0] + nr[1]);
    a.njb = fused ? (kPairBoth<T> ? 4 : 2) * jblocks(np) : 0;
    a.fchunk = a.nfreq;
    a.nchunk = 1;
    const size_t lds = std::max((size_t)a.nfreq * (sizeof(double) + sizeof(T)),
                                fused ? jlds_bytes(kPairGroup, sizeof(T)) : 0);
    for (; step < nz; step += 2, ++launch) {
      const int slot = (launch & 1) * 2;
      a.jsame = 0;
      for (int i = 0; i < A.njprev[0] && nr[0] > 0 && nr[1] > 0; ++i)
        for (int j = 0; j < A.njprev[1]; ++j) a.jsame |= A.jp[0][i].off == A.jp[1][j].off;
      T* next[2];
      for (int m = m0; m < m1; ++m) {
        const int k = kb[m] + up[m] * step, s = up[m];
        next[m] = kept(m, k + s, r0[m]);
        if (!next[m]) next[m] = state[launch & 1] + soff[m];
        set(a.h[at[m]], m, k, prev[m], kept(m, k, r0[m]), slot);
        set(A.n[at[m]], m, k + s, nullptr, next[m], slot + 1);
      }
      hipLaunchKernelGGL(k_sweep_pair<T>, dim3(a.nstep + a.njb), dim3(kPairThreads), lds, st, A);
      if ((e = check_launch("sweep_pair"))) return e;
      for (int m = m0; m < m1; ++m) {
        const int k = kb[m] + up[m] * step;
        A.jp[at[m]][0] = {a.h[at[m]].jpart, (size_t)k * np};
        A.jp[at[m]][1] = {A.n[at[m]].jpart, (size_t)(k + up[m]) * np};
        A.njprev[at[m]] = 2;
        prev[m] = next[m];
      }
      if (jkq && !fused && (e = reduce())) return e;
    }
    if (fused) return reduce();   // the last launch's planes
    return PORTA_OK;
  };
  if (P.pair && interp == PORTA_INTERP_BILINEAR)
    return walk_batches(q, o, P, jkq == nullptr, walk_pairs);
  return walk_batches(q, o, P, jkq == nullptr, walk);
}

// ---------------------------------------------------------------------------
// Adjoint of the sweep of the upward rays
// ---------------------------------------------------------------------------
template <class T>
int forward_plane(const porta_grid* g, const porta_quad* q, const porta_fields* f,
                  const porta_options* o, int interp, char* ws, const Layout& L, Geometry& geo,
                  int k, const T* prev, T* next, int ray0, int nrb, int block, hipStream_t st) {
  const int rc = geo.need(ray0, nrb, k, 1, st);
  if (rc) return rc;
  PlaneArgs<T> a = plane_args<T>(g, q, f, o, ws, L, geo);
  set_chunks(a, adjoint_chunks<T>((int64_t)a.ntile * nrb, q->nfreq, interp), nrb);
  HemiArgs<T>& h = a.h[0];
  set_plane(h, g, k, 1);
  h.iprev = prev;
  h.inext = next;
  h.ray0 = ray0;
  h.nrb = nrb;
  h.ibound = (T)f->i_bottom;
  return launch_plane<T>(a, 4, interp, block, st);
}

// Nodes per block of the gather: 64, whole wavefronts of neighbouring nodes, or 16 and four
// times the ray groups where a plane has too few nodes.  A plane takes, with 64 and 16 nodes, in
// the bilinear mode 22.0 and 29.3 us at 64x64 nodes, 9.5 and 10.2 us at 37x30, and in the
// 9-point mode, where a ray costs far more, 37.5 and 23.7 us at 24x24.  Bilinear planes of
// one node per thread from 24576 nodes: 16 rays in FP32 take 24 and 39 us at 192x176 with and
// without, 21 and 20 at 128x128.  9-point planes so with few rays, which leave groups of rays
// idle: adjoints of 8 planes, 4 frequencies, with and without, FP64 128x128, 1 and 2 rays 0.77 and
// 1.07 ms, 0.91 and 0.97; 200x200, 1, 2 and 4 rays 0.79 and 1.28, 1.15 and 1.59, 1.91 and 2.20;
// 300x300, 12 rays 11.6 and 12.1, 16 rays alike; FP32 200x200, 1, 2 and 4 rays 0.68 and 1.05, 0.93
// and 1.22, 1.54 and 1.58; 8 rays 0.92 to 0.98 times as fast.
template <class T>
void launch_gather(const GatherArgs<T>& b, bool bez, hipStream_t st) {
  const dim3 blk(256), one((b.np + 255) / 256, 4);
  if (!bez && b.nchunk == 1 && b.np >= kCus * 96) {
    hipLaunchKernelGGL((k_adjoint_gather_wide<T, 0>), one, blk, 0, st, b);
    return;
  }
  if (bez && (b.nrb <= 2 ? b.np >= kCus * 64
                         : b.nrb <= (sizeof(T) == 8 ? 12 : 4) && b.np >= kCus * 144)) {
    hipLaunchKernelGGL((k_adjoint_gather_wide<T, 1>), one, blk, 0, st, b);
    return;
  }
  const bool wide = b.np >= kCus * (bez ? 16 : 4);
  const unsigned n = (unsigned)((b.np + (wide ? 63 : 15)) / (wide ? 64 : 16));
  if (bez && wide)
    hipLaunchKernelGGL((k_adjoint_gather<T, 1, 64>), dim3(n, kGatherParts), blk, 0, st, b);
  else if (bez)
    hipLaunchKernelGGL((k_adjoint_gather<T, 1, 16>), dim3(n, kGatherParts), blk, 0, st, b);
  else if (wide)
    hipLaunchKernelGGL((k_adjoint_gather<T, 0, 64>), dim3(n, kGatherParts), blk, 0, st, b);
  else
    hipLaunchKernelGGL((k_adjoint_gather<T, 0, 16>), dim3(n, kGatherParts), blk, 0, st, b);
}

template <class T>
int adjoint_impl(const porta_grid* g, const porta_quad* q, const porta_fields* f,
                 const porta_options* o, int interp, const T* seed, const T* ext_ck, int C, T* gk,
                 T* gpm, T* ge, char* ws, const Layout& L, hipStream_t st) {
  int rc;
  if (!ext_ck) C = L.stride;
  Geometry geo;
  if ((rc = prepare_tables<T>(ws, L, g, q, f->w2, interp, &geo, st))) return rc;
  const int nx = g->nx, ny = g->ny, nz = g->nz, np = nx * ny;
  const size_t N = (size_t)np * nz;
  double* grad = reinterpret_cast<double*>(ws + L.grad);
  if ((rc = fill(grad, 13 * N, 0.0, st))) return rc;
  const int nrb_max = ray_batch(q, o);
  const int block = plane_block(g, o);
  if (block % 64 != 0 || block > 256) return fail(PORTA_EINVAL, "block must be 64, 128, 192 or 256");
  const int ntile = (int)plane_tiles(g, o);
  const size_t pe = L.plane / sizeof(T);   // elements of one plane state
  T* ck = reinterpret_cast<T*>(ws + L.ck);
  T* slots = reinterpret_cast<T*>(ws + L.slots);
  T* lam[2] = {reinterpret_cast<T*>(ws + L.lamA), reinterpret_cast<T*>(ws + L.lamB)};
  // forward state of plane k of the current batch: the boundary (nullptr), a
  // checkpoint (own or the caller's, rays contiguous in both), or a recompute slot
  int r0 = 0, up_lo, up_hi;
  hemi_range(q, o, 0, up_lo, up_hi);
  auto plane = [&](int k) -> T* {
    if (k == 0) return nullptr;
    if (is_checkpoint(k, nz, C)) {
      if (ext_ck)
        return const_cast<T*>(ext_ck) +
               ((size_t)(k / C - 1) * (up_hi - up_lo) + (r0 - up_lo)) * q->nfreq * np * 4;
      return ck + (size_t)(k / C - 1) * pe;
    }
    return slots + (size_t)((k - 1) % C) * pe;
  };
  for (r0 = up_lo; r0 < up_hi; r0 += nrb_max) {
    const int nrb = std::min(nrb_max, up_hi - r0);
    // the workspace has room for the chunks of a full batch
    const int want = std::min(adjoint_chunks<T>((int64_t)ntile * nrb, q->nfreq, interp),
                              nrb_max * freq_chunks((int64_t)ntile * nrb_max, q->nfreq) / nrb);
    const int fchunk = (q->nfreq + want - 1) / want, nchunk = (q->nfreq + fchunk - 1) / fchunk;
    const dim3 agrid((unsigned)(ntile * nrb * nchunk));
    const size_t lds_adj = (size_t)fchunk * sizeof(T);
    // forward pass up to the last checkpoint plane, keeping every C-th plane (unless
    // the sweep already kept them); the planes above it are recomputed with the top
    // segment
    if (!ext_ck)
      for (int k = 1; k <= C * checkpoint_count(nz, C); ++k)
        if ((rc = forward_plane<T>(g, q, f, o, interp, ws, L, geo, k, plane(k - 1), plane(k), r0,
                                   nrb, block, st)))
          return rc;
    // reverse pass, one segment between checkpoints at a time
    const T* lam_next = nullptr;
    int cur = 0;
    for (int khi = nz - 1; khi >= 1;) {
      const int s0 = C * ((khi - 1) / C);
      // the adjoint of plane k reads the forward state of plane k-1 only, so the top
      // plane of a segment needs no state
      for (int k = s0 + 1; k < khi; ++k)
        if (!is_checkpoint(k, nz, C))
          if ((rc = forward_plane<T>(g, q, f, o, interp, ws, L, geo, k, plane(k - 1), plane(k), r0,
                                     nrb, block, st)))
            return rc;
      for (int k = khi; k > s0; --k) {
        if ((rc = geo.need(r0, nrb, k, -1, st))) return rc;
        AdjArgs<T> a;
        a.kappa = static_cast<const T*>(f->kappa);
        a.prop = static_cast<const T*>(f->propmat);
        a.emis = static_cast<const T*>(f->emis);
        a.rays = reinterpret_cast<const RayConsts*>(ws + L.rays);
        geo.set(a);
        a.phi = reinterpret_cast<const T*>(ws + L.phiT);
        a.iprev = plane(k - 1);
        a.lam_next = lam_next;
        a.seed = seed + (size_t)r0 * q->nfreq * np * 4;
        a.lam_cur = (k - 1 >= 1) ? lam[cur] : nullptr;
        a.g_o = reinterpret_cast<T*>(ws + L.go);
        a.g_m = reinterpret_cast<T*>(ws + L.gm);
        a.g_p = reinterpret_cast<T*>(ws + L.gp);
        a.N = N;
        a.nx = nx;
        a.ny = ny;
        a.np = np;
        a.nfreq = q->nfreq;
        a.ntile = ntile;
        a.fchunk = fchunk;
        a.nchunk = nchunk;
        a.kO = k;
        a.kM = k - 1;
        a.kP = (k == nz - 1) ? -1 : k + 1;
        a.ray0 = r0;
        a.xcd_remap = xcd_chunk(o);
        a.parabolic = parabolic_of(o);
        a.ibound = (T)f->i_bottom;
        const bool bez = interp == PORTA_INTERP_BEZIER2D;
        if (bez && lam_next) {
          // the adjoint of the Stokes vectors of plane k, gathered through the transposed
          // 9-point stencils of plane k + 1, into the buffer the adjoint of plane k then
          // reads as its seed and overwrites, node by node, with its own output
          TGatherArgs<T> t;
          t.icur = plane(k);
          t.lam_next = lam_next;
          t.out = lam[cur];
          t.geom = a.geom;
          t.nx = nx;
          t.ny = ny;
          t.nz = a.nz;
          t.np = np;
          t.nfreq = q->nfreq;
          t.kO = k;
          t.ray0 = r0;
          constexpr int TX = TGTile<T>::X, TY = TGTile<T>::Y;
          const int tx = (nx + TX - 1) / TX, ty = (ny + TY - 1) / TY;
          // (at most 65535 in a grid's z)
          const int tc = std::min(freq_chunks((int64_t)tx * ty * nrb, q->nfreq),
                                  std::max(1, 65535 / nrb));
          t.fchunk = (q->nfreq + tc - 1) / tc;
          t.nchunk = (q->nfreq + t.fchunk - 1) / t.fchunk;
          hipLaunchKernelGGL(k_bez9_tgather<T>, dim3(tx, ty, nrb * t.nchunk), dim3(TX * TY), 0,
                             st, t);
          if ((rc = check_launch("bez9_tgather"))) return rc;
          a.lam_next = nullptr;
          a.seed = lam[cur];
          a.lam_cur = (k - 1 >= 1) ? lam[cur] : nullptr;
        }
        if (bez)
          hipLaunchKernelGGL((k_adjoint_plane<T, 1>), agrid, dim3(block), lds_adj, st, a);
        else
          hipLaunchKernelGGL((k_adjoint_plane<T, 0>), agrid, dim3(block), lds_adj, st, a);
        if ((rc = check_launch("adjoint_plane"))) return rc;
        GatherArgs<T> b;
        b.g_o = a.g_o;
        b.g_m = a.g_m;
        b.g_p = a.g_p;
        b.kappa = a.kappa;
        b.prop = a.prop;
        b.emis = a.emis;
        b.geom = a.geom;
        b.grad = grad;
        b.N = N;
        b.nx = nx;
        b.ny = ny;
        b.nz = a.nz;
        b.np = np;
        b.kO = a.kO;
        b.kM = a.kM;
        b.kP = a.kP;
        b.ray0 = r0;
        b.nrb = nrb;
        b.nchunk = nchunk;
        launch_gather<T>(b, bez, st);
        if ((rc = check_launch("adjoint_gather"))) return rc;
        lam_next = a.lam_cur;
        cur ^= 1;
      }
      khi = s0;
    }
  }
  const size_t blocks = std::min<size_t>((N + 255) / 256, 65536);
  hipLaunchKernelGGL(k_grad_out<T>, dim3((unsigned)blocks), dim3(256), 0, st, grad, N, gk, gpm, ge);
  return check_launch("grad_out");
}


// ---------------------------------------------------------------------------
// Static scratch of porta_fs_sweep_noalloc: one array per device, the workspace of
// that entry point.  Host code never uses the symbol itself as an address: the
// device address is looked up once per device (with that device current) and kept.
// ---------------------------------------------------------------------------
constexpr int kMaxDevices = 64;

std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of the current device's scratch array.
int scratch_address(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0)
    return fail(PORTA_EDEVICE, "no current HIP device");
  if (dev >= kMaxDevices) return fail(PORTA_EUNSUPPORTED, "device index %d >= %d", dev, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
      return fail(PORTA_EDEVICE, "hipGetSymbolAddress(scratch) on device %d: %s", dev,
                  hipGetErrorString(e));
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return PORTA_OK;
}

// Validation and launch of a forward sweep.  With use_scratch the workspace is this
// device's static scratch array instead of the caller's buffer.
int sweep_entry(const porta_grid* grid, const porta_quad* quad, const porta_fields* fields,
                int prec, int interp, const porta_options* opts, double* jkq, int accumulate,
                void* i_top, void* checkpoints, size_t ck_bytes, int checkpoint_stride,
                void* workspace, size_t ws_bytes, bool use_scratch, void* stream) {
  int rc;
  if ((rc = validate_grid(grid)) || (rc = validate_quad(quad)) || (rc = validate_prec(prec)) ||
      (rc = validate_interp(interp)))
    return rc;
  if (!fields || !fields->kappa || !fields->propmat || !fields->emis)
    return fail(PORTA_EINVAL, "fields and their arrays must not be NULL");
  if (!std::isfinite(fields->i_bottom) || !std::isfinite(fields->w2))
    return fail(PORTA_EINVAL, "i_bottom and w2 must be finite");
  if ((rc = validate_options(opts)) || (rc = validate_rays(quad, opts))) return rc;
  if (nstokes(opts) == 1 && interp != PORTA_INTERP_BILINEAR)
    return fail(PORTA_EUNSUPPORTED, "the intensity-only sweep interpolates bilinearly only");
  if (nstokes(opts) == 1 && checkpoints)
    return fail(PORTA_EUNSUPPORTED, "checkpoints are for the Stokes-vector sweep");
  if (faces_of(opts)) {
    if (nstokes(opts) == 1 || interp != PORTA_INTERP_BILINEAR || checkpoints)
      return fail(PORTA_EUNSUPPORTED,
                  "faces = 1 is for the bilinear Stokes-vector sweep without checkpoints");
    if (std::max(grid->nx, grid->ny) > kFacesMaxLanes)
      return fail(PORTA_EUNSUPPORTED, "faces = 1 needs nx, ny <= %d", kFacesMaxLanes);
    const size_t want = opts->faces_chunk > 0 ? std::min(opts->faces_chunk, quad->nfreq) : 1;
    if (want > faces_fit(grid, quad, prec))
      return fail(PORTA_EUNSUPPORTED, "faces = 1: the LDS of a block has no room for %s",
                  opts->faces_chunk > 0 ? "faces_chunk frequencies" : "one frequency");
  }
  if (checkpoints && (checkpoint_stride < 1 || checkpoint_stride > grid->nz - 1))
    return fail(PORTA_EINVAL, "checkpoint_stride must be in 1..nz-1");
  if (checkpoints) {
    const size_t need = checkpoint_bytes(grid, quad, prec, checkpoint_stride, opts);
    if (ck_bytes < need)
      return fail(PORTA_ENOMEM, "checkpoint buffer of %zu bytes is smaller than the %zu required",
                  ck_bytes, need);
  }
  if (!use_scratch && !workspace) return fail(PORTA_EINVAL, "workspace is NULL");
  SweepPlan plan = sweep_plan(grid, quad, prec, opts);
  Layout L = sweep_layout(grid, quad, prec, opts, plan);
  if (use_scratch) {
    const size_t need = scratch_need(grid, quad, prec, opts);
    if (need > kScratchLimit)
      return fail(PORTA_ENOMEM,
                  "this sweep needs %zu bytes of workspace; the static scratch holds %zu "
                  "(use a smaller opts->ray_batch, or porta_fs_sweep)",
                  need, kScratchLimit);
    // the cut that fits: the usual one, the plain one, or that with fewer rays in turn, whose
    // window of the rays' geometry takes what is left
    if (L.total > kScratchBytes) {
      int nrb = plan.nrb;
      do {
        plan = least_plan(grid, nrb);
        L = sweep_layout(grid, quad, prec, opts, plan);
      } while (L.total > kScratchBytes && --nrb > 0);
      if (L.total > kScratchBytes)
        return fail(PORTA_ENOMEM, "this sweep does not fit the static scratch of %zu bytes",
                    kScratchBytes);
      const size_t layer = plan.nrb * kGeomEntry + sizeof(double), align = 2 * kAlign;
      if (L.window > 0 && kScratchBytes - L.total > align)
        plan.window = (int)std::min<size_t>(
            grid->nz - 1, L.window + (kScratchBytes - L.total - align) / layer);
      L = sweep_layout(grid, quad, prec, opts, plan);
    }
    if ((rc = scratch_address(&workspace))) return rc;
    ws_bytes = kScratchBytes;
  }
  if (ws_bytes < L.total)
    return fail(PORTA_ENOMEM, "workspace of %zu bytes is smaller than the %zu required", ws_bytes,
                L.total);
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  if (opts && opts->check_inputs &&
      (rc = (prec == PORTA_F64) ? check_inputs<double>(grid, fields, ws, L, st)
                                : check_inputs<float>(grid, fields, ws, L, st)))
    return rc;
  if (prec == PORTA_F64)
    return sweep_impl<double>(grid, quad, fields, interp, opts, jkq, accumulate,
                              static_cast<double*>(i_top), static_cast<double*>(checkpoints),
                              checkpoint_stride, ws, plan, L, st);
  return sweep_impl<float>(grid, quad, fields, interp, opts, jkq, accumulate,
                           static_cast<float*>(i_top),
                           static_cast<float*>(checkpoints), checkpoint_stride, ws, plan, L, st);
}

}  // namespace

extern "C" {

const char* porta_version(void) { return "porta-mi355x 0.1.0 (gfx950)"; }

const char* porta_last_error(void) { return g_last_error.c_str(); }

const char* porta_strerror(int status) {
  switch (status) {
    case PORTA_OK: return "success";
    case PORTA_EINVAL: return "invalid argument";
    case PORTA_EUNSUPPORTED: return "unsupported combination of arguments";
    case PORTA_ENOMEM: return "workspace too small";
    case PORTA_EDEVICE: return "HIP device error";
    case PORTA_ENONFINITE: return "non-finite transfer coefficient or eta_I <= 0";
    default: return "unknown status";
  }
}

size_t porta_workspace_size(const porta_grid* grid, const porta_quad* quad, int prec, int kind,
                            int checkpoint_stride, const porta_options* opts) {
  if (validate_prec(prec)) return 0;
  switch (kind) {
    case PORTA_WS_SWEEP:
      if (validate_grid(grid) || validate_quad(quad)) return 0;
      return sweep_bytes(grid, quad, prec, opts);
    case PORTA_WS_ADJOINT:
    case PORTA_WS_ADJOINT_CKPT:
      if (validate_grid(grid) || validate_quad(quad) || checkpoint_stride < 1 ||
          checkpoint_stride > grid->nz - 1)
        return 0;
      return adjoint_bytes(grid, quad, prec, checkpoint_stride, opts, kind == PORTA_WS_ADJOINT);
    case PORTA_WS_JKQ:
      if (validate_quad(quad)) return 0;
      return tables_layout(quad, prec, 0).total;
    case PORTA_WS_SEE: {
      if (!grid || grid->nx < 1 || grid->ny < 1 || grid->nz < 1) return 0;
      const size_t n = (size_t)grid->nx * grid->ny * grid->nz;
      return align_up(sizeof(double) * ((n + 255) / 256));
    }
    default:
      fail(PORTA_EINVAL, "unknown workspace kind %d", kind);
      return 0;
  }
}

size_t porta_checkpoint_size(const porta_grid* grid, const porta_quad* quad, int prec,
                             int checkpoint_stride, const porta_options* opts) {
  if (validate_prec(prec) || validate_grid(grid) || validate_quad(quad) ||
      validate_options(opts) || validate_rays(quad, opts))
    return 0;
  if (checkpoint_stride < 1 || checkpoint_stride > grid->nz - 1) {
    fail(PORTA_EINVAL, "checkpoint_stride must be in 1..nz-1");
    return 0;
  }
  return checkpoint_bytes(grid, quad, prec, checkpoint_stride, opts);
}

int porta_fs_sweep(const porta_grid* grid, const porta_quad* quad, const porta_fields* fields,
                   int prec, int interp, const porta_options* opts, double* jkq, int accumulate,
                   void* i_top, void* checkpoints, size_t ck_bytes, int checkpoint_stride,
                   void* workspace, size_t ws_bytes, void* stream) {
  return sweep_entry(grid, quad, fields, prec, interp, opts, jkq, accumulate, i_top, checkpoints,
                     ck_bytes, checkpoint_stride, workspace, ws_bytes, false, stream);
}

int porta_fs_sweep_noalloc(const porta_grid* grid, const porta_quad* quad,
                           const porta_fields* fields, int prec, int interp,
                           const porta_options* opts, double* jkq, int accumulate, void* i_top,
                           void* stream) {
  return sweep_entry(grid, quad, fields, prec, interp, opts, jkq, accumulate, i_top, nullptr, 0,
                     0, nullptr, 0, true, stream);
}

int porta_jkq_accumulate(const porta_grid* grid, const porta_quad* quad, int ray0, int nray,
                         int f0, int nf, const void* stokes, const void* lambda_star, int prec,
                         double* jkq, void* workspace, size_t ws_bytes, void* stream) {
  int rc;
  if ((rc = validate_grid(grid)) || (rc = validate_quad(quad)) || (rc = validate_prec(prec)))
    return rc;
  const int nrays = 2 * quad->nmu * quad->nchi;
  if (ray0 < 0 || nray < 0 || ray0 + nray > nrays)
    return fail(PORTA_EINVAL, "ray range [%d, %d) outside [0, %d)", ray0, ray0 + nray, nrays);
  if (f0 < 0 || nf < 0 || f0 + nf > quad->nfreq)
    return fail(PORTA_EINVAL, "frequency range [%d, %d) outside [0, %d)", f0, f0 + nf,
                quad->nfreq);
  if (!stokes || !jkq) return fail(PORTA_EINVAL, "stokes and jkq must not be NULL");
  if (!workspace) return fail(PORTA_EINVAL, "workspace is NULL");
  const Layout L = tables_layout(quad, prec, 0);
  if (ws_bytes < L.total)
    return fail(PORTA_ENOMEM, "workspace of %zu bytes is smaller than the %zu required", ws_bytes,
                L.total);
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  const size_t N = (size_t)grid->nx * grid->ny * grid->nz;
  if (nray == 0 || nf == 0) return PORTA_OK;
  const dim3 grd((unsigned)((N + 255) / 256)), blk(256);
  if (prec == PORTA_F64) {
    if ((rc = prepare_tables<double>(ws, L, nullptr, quad, 1.0, 0, nullptr, st))) return rc;
    hipLaunchKernelGGL(k_jkq_accumulate<double>, grd, blk, 0, st, jkq,
                       static_cast<const double*>(stokes), static_cast<const double*>(lambda_star),
                       reinterpret_cast<const RayConsts*>(ws + L.rays),
                       reinterpret_cast<const double*>(ws + L.wn), ray0, nray, f0, nf, N);
  } else {
    if ((rc = prepare_tables<float>(ws, L, nullptr, quad, 1.0, 0, nullptr, st))) return rc;
    hipLaunchKernelGGL(k_jkq_accumulate<float>, grd, blk, 0, st, jkq,
                       static_cast<const float*>(stokes), static_cast<const float*>(lambda_star),
                       reinterpret_cast<const RayConsts*>(ws + L.rays),
                       reinterpret_cast<const double*>(ws + L.wn), ray0, nray, f0, nf, N);
  }
  return check_launch("jkq_accumulate");
}

int porta_fs_adjoint(const porta_grid* grid, const porta_quad* quad, const porta_fields* fields,
                     int prec, int interp, const porta_options* opts, const void* dl_ditop,
                     const void* checkpoints, size_t ck_bytes, int checkpoint_stride,
                     void* g_kappa, void* g_propmat, void* g_emis, void* workspace,
                     size_t ws_bytes, void* stream) {
  int rc;
  if ((rc = validate_grid(grid)) || (rc = validate_quad(quad)) || (rc = validate_prec(prec)) ||
      (rc = validate_interp(interp)))
    return rc;
  if (!fields || !fields->kappa || !fields->propmat || !fields->emis)
    return fail(PORTA_EINVAL, "fields and their arrays must not be NULL");
  if (!dl_ditop || !g_kappa || !g_propmat || !g_emis)
    return fail(PORTA_EINVAL, "seed and gradient arrays must not be NULL");
  if (checkpoint_stride < 1 || checkpoint_stride > grid->nz - 1)
    return fail(PORTA_EINVAL, "checkpoint_stride must be in 1..nz-1");
  if ((rc = validate_options(opts)) || (rc = validate_rays(quad, opts))) return rc;
  if (nstokes(opts) == 1)
    return fail(PORTA_EUNSUPPORTED, "the adjoint is for the Stokes-vector sweep");
  if (faces_of(opts))
    return fail(PORTA_EUNSUPPORTED, "the adjoint differentiates the plane-hop sweep (faces = 0)");
  if (checkpoints) {
    const size_t need = checkpoint_bytes(grid, quad, prec, checkpoint_stride, opts);
    if (ck_bytes < need)
      return fail(PORTA_ENOMEM, "checkpoint buffer of %zu bytes is smaller than the %zu required",
                  ck_bytes, need);
  }
  if (!workspace) return fail(PORTA_EINVAL, "workspace is NULL");
  const Layout L = adjoint_layout(grid, quad, prec, checkpoint_stride, opts, !checkpoints,
                                  (size_t)ray_batch(quad, opts));
  if (ws_bytes < L.total)
    return fail(PORTA_ENOMEM, "workspace of %zu bytes is smaller than the %zu required", ws_bytes,
                L.total);
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  if (opts && opts->check_inputs &&
      (rc = (prec == PORTA_F64) ? check_inputs<double>(grid, fields, ws, L, st)
                                : check_inputs<float>(grid, fields, ws, L, st)))
    return rc;
  if (prec == PORTA_F64)
    return adjoint_impl<double>(grid, quad, fields, opts, interp,
                                static_cast<const double*>(dl_ditop),
                                static_cast<const double*>(checkpoints), checkpoint_stride,
                                static_cast<double*>(g_kappa), static_cast<double*>(g_propmat),
                                static_cast<double*>(g_emis), ws, L, st);
  return adjoint_impl<float>(grid, quad, fields, opts, interp,
                             static_cast<const float*>(dl_ditop),
                             static_cast<const float*>(checkpoints), checkpoint_stride,
                             static_cast<float*>(g_kappa), static_cast<float*>(g_propmat),
                             static_cast<float*>(g_emis), ws, L, st);
}

}  // extern "C"
