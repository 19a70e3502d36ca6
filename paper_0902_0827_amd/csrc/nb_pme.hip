// Reciprocal part of the Ewald sum by smooth particle-mesh Ewald (ACEMD paper, section 3:
// the long-range electrostatics are PME with fourth-order interpolation; the method is
// that of Essmann et al., J. Chem. Phys. 103, 8577 (1995)).  With u_a = K_a x_a / L_a
// the scaled fractional coordinates and M_4 the cubic cardinal B-spline:
//
//   Q(k)   = sum_i q_i prod_a M_4(u_ai - k_a)           (periodic in k)
//   E      = k_e/(2 pi V) sum_{m != 0} C(m) |FFT(Q)(m)|^2,
//   C(m)   = exp(-pi^2 m^2/beta^2)/m^2 prod_a 9/(2 + cos(2 pi m_a/K_a))^2
//   phi    = dE/dQ = k_e/(pi V) IFFT(C FFT(Q))          (unnormalised inverse)
//   F_i    = -q_i sum_k phi(k) grad_i prod_a M_4(u_ai - k_a)
//   W_ab   = sum_m E_m [delta_ab - 2 (1 + pi^2 m^2/beta^2) m_a m_b / m^2].
//
// The factor 9/(2 + cos t)^2 is |b(m)|^2 for order 4: the Euler exponential spline's
// denominator 1/6 + (2/3) e^{it} + (1/6) e^{2it} has modulus (2 + cos t)/3.
//
// All arithmetic is FP64 (positions and charges of either precision are promoted).  In
// order on the caller's stream, every system of a batch in the same launches:
//
//   k_pme_bin      per 1024 atoms: their scaled coordinates and charges, sorted by the
//                  x-plane they start in (a counting sort in LDS; left out where the grid is
//                  too coarse to hold them); three more workgroups write the tables of the FFTs;
//   k_pme_rows_fwd one workgroup per (system, x, block of y rows): the rows' charges summed
//                  in LDS from the atoms that touch them, then their real FFTs along z in
//                  place, and the half spectra stored by z frequency;
//   k_pme_slab     one workgroup per (system, z frequency): the FFTs along y and x in LDS,
//                  C(m) with the energy and virial terms, and the inverse FFTs;
//   k_pme_rows_inv per (system, x, block of y rows): the inverse FFT along z, giving phi;
//   k_pme_gather   8 lanes per atom: its force from phi and the spline derivatives; its
//                  last workgroups sum each system's energy and virial partials in order.
//
// Between the kernels the spectrum crosses memory twice instead of eight times, and nine
// launches are five.  Measured with energy and virial, MI355X: 63.2 -> 45.0 us per call for
// 23.6k atoms at 64^3, 224 -> 109 us for 24 systems (293k atoms) at 48^3.  (x-planes
// transformed whole, with a third kernel for the x lines, took 69 and 255 us: one system
// then has 64 workgroups, all of whose LDS additions queue on 64 CUs.)
// These take grids whose sizes have no prime factor above 7 and whose (x, y) planes fit in
// LDS (pme_grid below).  Other grids go through hipFFT, which moves the grid through memory
// between every two steps: k_pme_spread_planes (or k_pme_zero and k_pme_spread), D2Z,
// k_pme_convolve, Z2D, k_pme_gather.
// The grid additions of the spread (LDS or global atomics) are the only ones whose order
// varies from run to run.
#include <hipfft/hipfft.h>

#include <algorithm>
#include <cstring>
#include <map>
#include <mutex>
#include <tuple>
#include <type_traits>
#include <vector>

#include "nb_internal.h"
#include "nb_pair_common.h"
#include "nb_pme.h"
#include "nb_pme_fft.h"

namespace nb {

namespace {

constexpr double kPi = 3.14159265358979323846;
constexpr int kMinGrid = 4;     // the spline's four points must be distinct grid points
constexpr int kMaxGrid = 1024;

struct PmeSys {
  double L[3];
  double invL[3];
  double a;       // pi^2 / beta^2
  double escale;  // k_e / (2 pi V)
  int K[3];
  int H;  // K3/2 + 1: the half spectrum's last dimension
};

// Systems of one launch (at most kPmeChunk; a larger batch takes several launches per
// step).  Only what differs between systems travels here; the rest of PmeSys is formed on
// the device with the same IEEE operations as on the host (make_sys), so every system's
// constants are the ones a launch per system would have used.
// CAP: the systems it has room for.  A launch's arguments are written to the GPU by the host,
// and 2 kB of them take it about 3 us: one system travels in a descriptor of its own size.
constexpr int kPmeChunk = 32;
template <int CAP>
struct PmeBatch {
  static constexpr int kCap = CAP;
  int nsys;    // systems in this launch
  int first;   // batch index of its first system (grid and partial offsets)
  int K[3];
  double a;    // pi^2 / beta^2
  double ke;
  double L[CAP][3];
  double invL[CAP][3];
  int64_t a0[CAP];          // first atom of each system
  int32_t n[CAP];           // atoms of each system
  int32_t blk0[CAP + 1];    // first gather workgroup of each system (prefix sums)
  int32_t bin0[CAP + 1];    // first k_pme_bin workgroup of each system (whole batch)
};

// The same for a batch of more systems than travel in one launch's arguments, with the arrays in
// the workspace, written by k_pme_bin_table: one launch per step for all of them instead of one
// for each kPmeChunk, which took 7 us each (100 systems of 648 atoms on 20^3: 142 us with five
// launches for each 32, 122 through hipFFT, 77 with the table).
struct PmeTable {
  int nsys;   // systems in this launch
  int first;  // batch index of its first system
  int K[3];
  int wg0, wgs;  // gather workgroups of the systems before this launch's, and of its own
  double a, ke;
  double (*L)[3], (*invL)[3];
  int64_t *a0;
  int32_t *n, *blk0, *bin0;
};

// System k of the launch.
template <typename PB>
__host__ __device__ inline PmeSys make_sys(const PB &pb, int k) {
  PmeSys ps;
  for (int d = 0; d < 3; ++d) {
    ps.L[d] = pb.L[k][d];
    ps.invL[d] = pb.invL[k][d];
    ps.K[d] = pb.K[d];
  }
  ps.H = ps.K[2] / 2 + 1;
  ps.a = pb.a;
  ps.escale = pb.ke / (2.0 * kPi * ps.L[0] * ps.L[1] * ps.L[2]);
  return ps;
}

// The launch's system whose workgroups (prefix sums `first`) include wg: one load per lane
// and a ballot, instead of a walk whose every step waits for its own load.
template <int CAP>
__device__ inline int system_of_wg(const PmeBatch<CAP> &pb, const int32_t (&first)[CAP + 1], int wg) {
  if constexpr (CAP == 1) return 0;
  const int lane = static_cast<int>(threadIdx.x) & 63;
  return __builtin_amdgcn_readfirstlane(__popcll(__ballot(lane < pb.nsys && first[lane < pb.nsys ? lane : 0] <= wg)) - 1);
}
// (a table: a 64-way search, two rounds for 4,096 systems)
__device__ inline int system_of_wg(const PmeTable &pb, const int32_t *first, int wg) {
  int lo = 0, hi = pb.nsys - 1;  // the answer is in [lo, hi]
  const int lane = static_cast<int>(threadIdx.x) & 63;
  while (hi > lo) {
    const int step = (hi - lo + 64) >> 6, probe = lo + lane * step;
    const uint64_t m = __ballot(probe <= hi && first[probe <= hi ? probe : lo] <= wg);  // (lane 0 always)
    lo += (63 - __clzll(static_cast<long long>(m))) * step;
    hi = lo + step - 1 < hi ? lo + step - 1 : hi;
  }
  return __builtin_amdgcn_readfirstlane(lo);
}

// Gather workgroups of a launch, and those of the batch's systems before it.
template <int CAP>
__device__ inline int gather_wgs(const PmeBatch<CAP> &pb) { return pb.blk0[pb.nsys]; }
template <int CAP>
__device__ inline int gather_wg0(const PmeBatch<CAP> &) { return 0; }
__device__ inline int gather_wgs(const PmeTable &pb) { return pb.wgs; }
__device__ inline int gather_wg0(const PmeTable &pb) { return pb.wg0; }

inline size_t align256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

// Scaled coordinate u = K (x/L mod 1), in [0, K] for finite x.
__device__ inline double scaled_coord(double x, double invL, int K) {
  double f = x * invL;
  f -= floor(f);  // in [0, 1] for finite x
  return f * K;
}

// Grid cell of scaled coordinate u: base = floor(u) in [0, K), t = u - base.
__device__ inline void grid_cell(double u, int K, int *base_out, double *t_out) {
  int base = 0;
  double t;
  if (u >= 0.0 && u < K) {
    base = static_cast<int>(floor(u));
    t = u - base;
  } else if (u == K) {  // f rounded up to 1: the point K is the point 0
    t = 0.0;
  } else {  // non-finite coordinate: indices stay in range, the results are NaN
    t = u - u;
  }
  *base_out = base;
  *t_out = t;
}

// M_4(t + j) and dM_4/du there, j = 0..3, t in [0, 1).
__device__ inline void spline4(double t, double w[4], double dw[4]) {
  const double t2 = t * t, t3 = t2 * t, s = 1.0 - t;
  w[0] = t3 * (1.0 / 6.0);
  w[1] = (1.0 + 3.0 * t + 3.0 * t2 - 3.0 * t3) * (1.0 / 6.0);
  w[2] = (4.0 - 6.0 * t2 + 3.0 * t3) * (1.0 / 6.0);
  w[3] = s * s * s * (1.0 / 6.0);
  dw[0] = 0.5 * t2;
  dw[1] = 0.5 * (1.0 + 2.0 * t - 3.0 * t2);
  dw[2] = 0.5 * (3.0 * t2 - 4.0 * t);
  dw[3] = -0.5 * s * s;
}

// The four grid points k = base - j (mod K), j = 0..3, of coordinate x, with M_4(u - k)
// and dM_4/du at u - k = t + j, t = u - base in [0, 1).
__device__ inline void spline4(double x, double invL, int K, int idx[4], double w[4], double dw[4]) {
  int base;
  double t;
  grid_cell(scaled_coord(x, invL, K), K, &base, &t);
  spline4(t, w, dw);
#pragma unroll
  for (int j = 0; j < 4; ++j) idx[j] = base - j < 0 ? base - j + K : base - j;
}

__global__ void __launch_bounds__(kBlock) k_pme_zero(double *__restrict__ g, int64_t n) {
  for (int64_t e = blockIdx.x * static_cast<int64_t>(kBlock) + threadIdx.x; e < n;
       e += static_cast<int64_t>(gridDim.x) * kBlock)
    g[e] = 0.0;
}

// 16 lanes per atom, one per (x, y) row of its 4 x 4 x 4 footprint: each lane adds the
// row's four z points.  Lane t of the grid takes atom t / 16 and row (t / 4 % 4, t % 4).
constexpr int kLanesPerAtom = 16;

template <typename T>
__global__ void __launch_bounds__(kBlock) k_pme_spread(const T *__restrict__ pos, const T *__restrict__ charge, int n,
                                                       PmeSys ps, double *__restrict__ grid) {
  const int64_t t = blockIdx.x * static_cast<int64_t>(kBlock) + threadIdx.x;
  const int i = static_cast<int>(t / kLanesPerAtom);
  if (i >= n) return;
  const int a = static_cast<int>(t >> 2) & 3, b = static_cast<int>(t) & 3;
  int ix[4], iy[4], iz[4];
  double wx[4], wy[4], wz[4], d[4];
  spline4(static_cast<double>(pos[3 * i + 0]), ps.invL[0], ps.K[0], ix, wx, d);
  spline4(static_cast<double>(pos[3 * i + 1]), ps.invL[1], ps.K[1], iy, wy, d);
  spline4(static_cast<double>(pos[3 * i + 2]), ps.invL[2], ps.K[2], iz, wz, d);
  const double qab = static_cast<double>(charge[i]) * wx[a] * wy[b];
  double *row = grid + (static_cast<int64_t>(ix[a]) * ps.K[1] + iy[b]) * ps.K[2];
#pragma unroll
  for (int c = 0; c < 4; ++c) unsafeAtomicAdd(&row[iz[c]], qab * wz[c]);
}

// One workgroup per x-plane of the grid: it reads every atom, keeps those whose
// footprint covers its plane (four planes per atom) and adds their 4 x 4 (y, z) points
// with LDS atomics into the plane held in LDS, then stores the plane.  No global
// atomics and no clearing pass.  Used when a plane fits in kPlaneMaxPoints doubles.
constexpr int kPlaneBlock = 1024;
constexpr int kPlaneMaxPoints = 8192;  // 64 KB of LDS

template <typename T>
__global__ void __launch_bounds__(kPlaneBlock) k_pme_spread_planes(const T *__restrict__ pos_all,
                                                                   const T *__restrict__ charge_all,
                                                                   PmeBatch<kPmeChunk> pb, int64_t grid_points, double *__restrict__ grids) {
  extern __shared__ __align__(16) double plane[];
  // workgroup (system b of the launch, plane x)
  const int b = static_cast<int>(blockIdx.x) / pb.K[0];
  const int x = static_cast<int>(blockIdx.x) - b * pb.K[0];
  const PmeSys ps = make_sys(pb, b);
  const T *__restrict__ pos = pos_all + 3 * pb.a0[b];
  const T *__restrict__ charge = charge_all + pb.a0[b];
  const int n = pb.n[b];
  double *__restrict__ grid = grids + static_cast<int64_t>(pb.first + b) * grid_points;
  const int P = ps.K[1] * ps.K[2];
  for (int j = threadIdx.x; j < P; j += kPlaneBlock) plane[j] = 0.0;
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += kPlaneBlock) {
    int bx;
    double tx;
    grid_cell(scaled_coord(static_cast<double>(pos[3 * i + 0]), ps.invL[0], ps.K[0]), ps.K[0], &bx, &tx);
    int a = bx - x;  // the atom covers plane x as its point base - a (mod K), a in [0, 4)
    if (a < 0) a += ps.K[0];
    if (a >= 4) continue;
    const double s = 1.0 - tx;
    const double wa = a == 0 ? tx * tx * tx * (1.0 / 6.0)
                    : a == 1 ? (1.0 + 3.0 * tx + 3.0 * tx * tx - 3.0 * tx * tx * tx) * (1.0 / 6.0)
                    : a == 2 ? (4.0 - 6.0 * tx * tx + 3.0 * tx * tx * tx) * (1.0 / 6.0)
                             : s * s * s * (1.0 / 6.0);
    int iy[4], iz[4];
    double wy[4], wz[4], d[4];
    spline4(static_cast<double>(pos[3 * i + 1]), ps.invL[1], ps.K[1], iy, wy, d);
    spline4(static_cast<double>(pos[3 * i + 2]), ps.invL[2], ps.K[2], iz, wz, d);
    const double qa = static_cast<double>(charge[i]) * wa;
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int c = 0; c < 4; ++c) unsafeAtomicAdd(&plane[iy[b] * ps.K[2] + iz[c]], qa * wy[b] * wz[c]);
  }
  __syncthreads();
  double *out = grid + static_cast<int64_t>(x) * P;
  for (int j = threadIdx.x; j < P; j += kPlaneBlock) out[j] = plane[j];
}

// Signed reciprocal index of grid index i: i for i <= K/2, else i - K.
__device__ inline int signed_index(int i, int K) { return 2 * i <= K ? i : i - K; }

// (2 + cos(2 pi i / K))^2 / 9: the reciprocal of the order-4 spline factor |b(m)|^2
__device__ inline double inv_bmod2(int i, int K) {
  const double c = 2.0 + cospi(2.0 * static_cast<double>(i) / static_cast<double>(K));
  return c * c * (1.0 / 9.0);
}

// Adds one element's terms: em = its energy, m its wave vector, vf = 2 (1 + pi^2 m^2/beta^2)/m^2.
// The half spectrum holds each element and its conjugate partner (K - i mod K per
// dimension) once (pair), except in the planes iz = 0 and iz = K3/2, whose partners are
// elements of their own.  The partner has the same |F|^2 and m^2; its signed indices are -m
// except on a Nyquist index K/2, which stays +K/2: the off-diagonal terms of a pair double,
// or cancel when just one of their two indices is a Nyquist index (nx, ny; never z's).
__device__ inline void add_spec_terms(double em, const double (&m)[3], double vf, bool pair, bool nx, bool ny,
                                      double (&v)[kSymSums]) {
  const double e = pair ? 2.0 * em : em, g = e * vf;
  v[0] += e;
  v[1] += e - g * m[0] * m[0];
  v[4] += e - g * m[1] * m[1];
  v[6] += e - g * m[2] * m[2];
  v[2] -= pair && nx != ny ? 0.0 : g * m[0] * m[1];
  v[3] -= pair && nx ? 0.0 : g * m[0] * m[2];
  v[5] -= pair && ny ? 0.0 : g * m[1] * m[2];
}

// The workgroup's sums of v into its slot of the partials, [kSymSums][n_part_blocks].
__device__ inline void store_partials(const double (&v)[kSymSums], double (*red)[8], double *partials,
                                      int64_t n_part_blocks, int64_t blk) {
  const double t = block_sym_sum(v, red);
  if (threadIdx.x < kSymSums) partials[static_cast<int64_t>(threadIdx.x) * n_part_blocks + blk] = t;
}

__global__ void __launch_bounds__(kBlock) k_pme_convolve(double2 *__restrict__ specs, PmeBatch<kPmeChunk> pb,
                                                         int64_t n_spec,
                                                         double *__restrict__ partials_all, int64_t n_part_blocks) {
  __shared__ double red[kWaves][8];
  // workgroup (system b of the launch, block blk of its half spectrum)
  const int b = static_cast<int>(blockIdx.x / n_part_blocks);
  const int64_t blk = blockIdx.x - static_cast<int64_t>(b) * n_part_blocks;
  const PmeSys ps = make_sys(pb, b);
  double2 *__restrict__ spec = specs + static_cast<int64_t>(pb.first + b) * n_spec;
  const int64_t e = blk * kBlock + threadIdx.x;
  double v[kSymSums] = {0, 0, 0, 0, 0, 0, 0};
  if (e < n_spec) {
    const int iz = static_cast<int>(e % ps.H);
    const int64_t r = e / ps.H;
    const int iy = static_cast<int>(r % ps.K[1]);
    const int ix = static_cast<int>(r / ps.K[1]);
    const double m[3] = {signed_index(ix, ps.K[0]) * ps.invL[0], signed_index(iy, ps.K[1]) * ps.invL[1],
                         signed_index(iz, ps.K[2]) * ps.invL[2]};
    const double m2 = m[0] * m[0] + m[1] * m[1] + m[2] * m[2];
    double2 F = spec[e];
    if (m2 > 0.0) {
      const double inv_m2 = 1.0 / m2;
      const double C =
          exp(-ps.a * m2) * inv_m2 / (inv_bmod2(ix, ps.K[0]) * inv_bmod2(iy, ps.K[1]) * inv_bmod2(iz, ps.K[2]));
      add_spec_terms(ps.escale * C * (F.x * F.x + F.y * F.y), m, 2.0 * (1.0 + ps.a * m2) * inv_m2,
                     !(iz == 0 || 2 * iz == ps.K[2]), 2 * ix == ps.K[0], 2 * iy == ps.K[1], v);
      const double sc = 2.0 * ps.escale * C;  // k_e / (pi V) C
      F.x *= sc;
      F.y *= sc;
    } else {
      F.x = 0.0;
      F.y = 0.0;
    }
    spec[e] = F;
  }
  store_partials(v, red, partials_all + static_cast<int64_t>(pb.first + b) * kSymSums * n_part_blocks, n_part_blocks,
                 blk);
}

// ---- grids transformed here: bin, rows, slab ----

constexpr int kBinAtoms = 1024;   // atoms per k_pme_bin workgroup, one per thread
constexpr int kPhiPad = 3;        // copies of a row's last three values before it
constexpr size_t kPmeLdsMax = 150 * 1024;  // of the 160 KB of LDS per CU
constexpr int kCus = 256;                  // compute units of the MI355X

// One atom for the charge spreading: scaled coordinates and charge.
struct alignas(32) PmeAtom { double ux, uy, uz, q; };

// What the kernels of this section share.  The tables are in the workspace, written by
// k_pme_bin: for each dimension its K twiddles, |b(m)|^2 by frequency, and the frequency of
// each FFT position (for z instead the position of each frequency).
struct PmeGrid {
  FftShape f[3];
  int H;       // K3/2 + 1
  int pairs;   // row pairs of a k_pme_rows_* workgroup (an even number of rows, the last one padded)
  int blocks;  // its workgroups per x-plane
  int zs;      // LDS slots per row pair: K3, odd so that rows start in different banks
  int ys;      // LDS slots per x line of a slab: K2, odd for the same reason
  double2 *tw[3];
  double *bm[3];
  int32_t *at[3];
};

size_t rows_lds_bytes(const PmeGrid &g) {
  return 16 * (static_cast<size_t>(g.pairs) * g.zs + g.f[2].n) + 4 * static_cast<size_t>(g.f[2].n);
}
size_t slab_lds_bytes(const PmeGrid &g) {
  return 16 * (static_cast<size_t>(g.f[0].n) * g.ys + 2 * g.f[0].n + 2 * g.f[1].n);
}

// The workgroup's row pairs in LDS: rows 2j and 2j + 1 are the real and imaginary parts of
// complex line j, so that one complex transform does both; frequencies k and K3 - k of the
// line then hold the two rows' frequency k in their place.
struct RowsLds {
  double2 *buf;   // [pairs * zs]
  double2 *tw;    // [K3]
  int32_t *pos;   // [K3] position of each frequency
  __device__ RowsLds(double *lds, const PmeGrid &g) {
    buf = reinterpret_cast<double2 *>(lds);
    tw = buf + g.pairs * g.zs;
    pos = reinterpret_cast<int32_t *>(tw + g.f[2].n);
  }
  __device__ void tables(const PmeGrid &g) const {  // by the whole workgroup, no barrier
    for (int k = static_cast<int>(threadIdx.x); k < g.f[2].n; k += static_cast<int>(blockDim.x)) {
      tw[k] = g.tw[2][k];
      pos[k] = g.at[2][k];
    }
  }
};

template <typename T>
__device__ inline PmeAtom pme_atom(const T *__restrict__ pos, const T *__restrict__ charge, int64_t i,
                                   const PmeSys &ps) {
  return {scaled_coord(static_cast<double>(pos[3 * i + 0]), ps.invL[0], ps.K[0]),
          scaled_coord(static_cast<double>(pos[3 * i + 1]), ps.invL[1], ps.K[1]),
          scaled_coord(static_cast<double>(pos[3 * i + 2]), ps.invL[2], ps.K[2]), static_cast<double>(charge[i])};
}

// Scaled coordinates and charges of 1,024 atoms, sorted by the plane of their first x point
// (a counting sort in LDS; the order within a plane is arbitrary), and where each plane
// begins: [K1 + 1] offsets within the 1,024.  The rows kernel then reads, for its plane,
// one run of each 1,024 instead of testing every atom.  The last three workgroups of the
// batch's first launch write the tables instead, one dimension each.
template <typename T, int CAP>
__device__ inline void pme_bin(const T *__restrict__ pos, const T *__restrict__ charge, const PmeBatch<CAP> &pb,
                               const PmeGrid &g, PmeAtom *__restrict__ atoms, uint16_t *__restrict__ offs) {
  __shared__ int cnt[kMaxGrid + 1];
  __shared__ int tot[kBinAtoms / 64];
  const int t = static_cast<int>(threadIdx.x), lane = t & 63, wave = t >> 6;
  const int wg = static_cast<int>(blockIdx.x) + pb.bin0[0];  // numbered over the whole batch
  if (wg >= pb.bin0[pb.nsys]) {  // the tables of dimension d
    const int d = wg - pb.bin0[pb.nsys], n = d == 0 ? pb.K[0] : d == 1 ? pb.K[1] : pb.K[2];
    if (t < n) {
      const FftShape &shape = d == 0 ? g.f[0] : d == 1 ? g.f[1] : g.f[2];
      double2 *tw = d == 0 ? g.tw[0] : d == 1 ? g.tw[1] : g.tw[2];
      double *bm = d == 0 ? g.bm[0] : d == 1 ? g.bm[1] : g.bm[2];
      int32_t *at = d == 0 ? g.at[0] : d == 1 ? g.at[1] : g.at[2];
      double s, c;
      sincospi(2.0 * static_cast<double>(t) / static_cast<double>(n), &s, &c);
      tw[t] = make_double2(c, -s);
      bm[t] = 9.0 / ((2.0 + c) * (2.0 + c));
      const int f = shape.freq(t);
      at[d == 2 ? f : t] = d == 2 ? t : f;
    }
    return;
  }
  const int sb = system_of_wg(pb, pb.bin0, wg);
  const PmeSys ps = make_sys(pb, sb);
  const int first = (wg - pb.bin0[sb]) * kBinAtoms;
  const bool have = first + t < pb.n[sb];
  const int K = ps.K[0];
  for (int k = t; k <= K; k += kBinAtoms) cnt[k] = 0;
  PmeAtom at{0, 0, 0, 0};
  int bin = 0;
  if (have) {
    at = pme_atom(pos, charge, pb.a0[sb] + first + t, ps);
    double frac;
    grid_cell(at.ux, K, &bin, &frac);
  }
  __syncthreads();
  int slot = 0;
  if (have) slot = atomicAdd(&cnt[bin], 1);
  __syncthreads();
  // exclusive scan of the K <= 1024 counts, one per thread
  const int c = t < K ? cnt[t] : 0;
  int incl = c;
  for (int off = 1; off < 64; off <<= 1) {
    const int y = __shfl_up(incl, off, 64);
    if (lane >= off) incl += y;
  }
  if (lane == 63) tot[wave] = incl;
  __syncthreads();
  int before = 0;
  for (int k = 0; k < wave; ++k) before += tot[k];
  const int start = before + incl - c;
  uint16_t *out = offs + static_cast<int64_t>(wg) * (K + 1);
  if (t < K) {
    cnt[t] = start;
    out[t] = static_cast<uint16_t>(start);
    if (t == K - 1) out[K] = static_cast<uint16_t>(start + c);
  }
  __syncthreads();
  if (have) atoms[pb.a0[sb] + first + cnt[bin] + slot] = at;
}

template <typename T, int CAP>
__global__ void __launch_bounds__(kBinAtoms) k_pme_bin(const T *__restrict__ pos, const T *__restrict__ charge,
                                                       PmeBatch<CAP> pb, PmeGrid g, PmeAtom *__restrict__ atoms,
                                                       uint16_t *__restrict__ offs) {
  pme_bin<T, CAP>(pos, charge, pb, g, atoms, offs);
}

// The same for a batch with a table: the last workgroup writes this launch's systems into it.
template <typename T>
__global__ void __launch_bounds__(kBinAtoms) k_pme_bin_table(const T *__restrict__ pos, const T *__restrict__ charge,
                                                             PmeBatch<kPmeChunk> pb, PmeGrid g,
                                                             PmeAtom *__restrict__ atoms, uint16_t *__restrict__ offs,
                                                             PmeTable tab) {
  if (blockIdx.x + 1 < gridDim.x) {
    pme_bin<T, kPmeChunk>(pos, charge, pb, g, atoms, offs);
    return;
  }
  const int k = static_cast<int>(threadIdx.x), at = pb.first + k;
  if (k < pb.nsys) {
    for (int d = 0; d < 3; ++d) {
      tab.L[at][d] = pb.L[k][d];
      tab.invL[at][d] = pb.invL[k][d];
    }
    tab.a0[at] = pb.a0[k];
    tab.n[at] = pb.n[k];
  }
  if (k <= pb.nsys) {
    tab.blk0[at] = pb.blk0[k];
    tab.bin0[at] = pb.bin0[k];
  }
}

// Workgroup -> (system of the launch, x-plane, first row).
template <typename PB>
__device__ inline void rows_of(const PB &pb, const PmeGrid &g, int *b, int *x, int *y0) {
  const int wg = static_cast<int>(blockIdx.x), plane = wg / g.blocks;
  *y0 = (wg - plane * g.blocks) * 2 * g.pairs;
  *b = plane / pb.K[0];
  *x = plane - *b * pb.K[0];
}

// Rows [y0, y0 + 2 pairs) of plane x: charges, FFT along z, half spectra.  Bound by the
// rate of the FP64 LDS additions (16 per atom and plane, about 1.2 cycles each on a CU,
// whatever the lanes that share an instruction): several workgroups per plane where one
// system would otherwise leave CUs idle.
// atoms, offs: the binned atoms and where each plane's begin in each 1,024, or (T != PmeAtom) the
// caller's positions and charges.
template <typename T, typename U, typename PB>
__global__ void __launch_bounds__(kPlaneBlock) k_pme_rows_fwd(const T *__restrict__ atoms, const U *__restrict__ offs,
                                                              PB pb, PmeGrid g,
                                                              double2 *__restrict__ specs) {
  extern __shared__ __align__(16) double plane[];
  int b, x, y0;
  rows_of(pb, g, &b, &x, &y0);
  const int K1 = pb.K[0], K2 = pb.K[1], K3 = pb.K[2], rows = 2 * g.pairs;
  const RowsLds p(plane, g);
  const int t = static_cast<int>(threadIdx.x), lane = t & 63, wave = t >> 6;
  const int threads = static_cast<int>(blockDim.x), waves = threads >> 6;
  for (int k = t; k < g.pairs * g.zs; k += threads) p.buf[k] = make_double2(0.0, 0.0);
  p.tables(g);
  __syncthreads();
  // One atom's charges in the workgroup's rows of plane x.
  auto add = [&](const PmeAtom at) {
    int bx, by, bz;
    double fx, fy, fz, wx[4], wy[4], wz[4], d[4];
    grid_cell(at.uy, K2, &by, &fy);
    int r0 = by - y0;  // the atom's rows are by - i (mod K2), i in [0, 4)
    if (r0 < 0) r0 += K2;
    if (r0 >= rows + 3) return;
    grid_cell(at.ux, K1, &bx, &fx);
    grid_cell(at.uz, K3, &bz, &fz);
    int a = bx - x;  // the atom's point base - a (mod K1) is x
    if (a < 0) a += K1;
    spline4(fx, wx, d);
    spline4(fy, wy, d);
    spline4(fz, wz, d);
    const double qa = at.q * (a == 0 ? wx[0] : a == 1 ? wx[1] : a == 2 ? wx[2] : wx[3]);
    int iz[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) iz[j] = 2 * (bz - j < 0 ? bz - j + K3 : bz - j);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = r0 - i < 0 ? r0 - i + K2 : r0 - i;  // row within the workgroup's
      if (r >= rows) continue;
      double *row = plane + 2 * (r >> 1) * g.zs + (r & 1);
      const double qy = qa * wy[i];
#pragma unroll
      for (int j = 0; j < 4; ++j) unsafeAtomicAdd(&row[iz[j]], qy * wz[j]);
    }
  };
  if constexpr (std::is_same_v<T, PmeAtom>) {
    // Charges: plane x is touched by the atoms that start in x .. x + 3, one run (two where
    // that wraps) of each 1,024.  Each lane reads one such run's ends, 64 at a time; the waves
    // then take the runs' pieces of 64 atoms in turn (input sorted in space has most of a
    // plane's atoms in a few of the runs).
    const int hi = x + 4 < K1 ? x + 4 : K1, wrap = x + 4 > K1 ? x + 4 - K1 : 0;
    for (int c0 = pb.bin0[b]; c0 < pb.bin0[b + 1]; c0 += 64) {
      const int mine = c0 + lane;
      int my_s0 = 0, my_n0 = 0, my_n = 0;
      if (mine < pb.bin0[b + 1]) {
        const uint16_t *o = offs + static_cast<int64_t>(mine) * (K1 + 1);
        my_s0 = o[x];
        my_n0 = o[hi] - my_s0;
        my_n = my_n0 + (wrap ? o[wrap] : 0);
      }
      int pieces;
      const int upto = wave_excl_scan_int((my_n + 63) >> 6, &pieces);
      for (int piece = wave; piece < pieces; piece += waves) {
        // the run holding this piece: the last one that begins at or before it
        const int run = __popcll(__ballot(upto <= piece)) - 1;
        const int s0 = __shfl(my_s0, run, 64), n0 = __shfl(my_n0, run, 64), n = __shfl(my_n, run, 64);
        const int k = ((piece - __shfl(upto, run, 64)) << 6) + lane;
        if (k >= n) continue;
        const PmeAtom at =
            atoms[pb.a0[b] + static_cast<int64_t>(c0 - pb.bin0[b] + run) * kBinAtoms + (k < n0 ? s0 + k : k - n0)];
        add(at);
      }
    }
  } else {
    // every atom of the system, kept when it touches plane x
    const PmeSys ps = make_sys(pb, b);
    for (int i = t; i < pb.n[b]; i += threads) {
      const PmeAtom at = pme_atom(atoms, offs, pb.a0[b] + i, ps);
      int bx;
      double fx;
      grid_cell(at.ux, K1, &bx, &fx);
      if ((bx < x ? bx - x + K1 : bx - x) < 4) add(at);
    }
  }
  __syncthreads();
  fft_lines<false>([&](int l) { return [q = p.buf + l * g.zs](int e) { return q + e; }; }, g.pairs, g.f[2], p.tw);
  // the rows of each pair apart: A_k = (Z_k + conj Z_-k)/2, B_k = (Z_k - conj Z_-k)/2i
  double2 *out = specs + static_cast<int64_t>(pb.first + b) * g.H * K1 * K2 + static_cast<int64_t>(x) * K2 + y0;
  const float rr = __builtin_amdgcn_rcpf(static_cast<float>(rows));
  for (int u = t; u < rows * g.H; u += threads) {
    const int k = small_div(u, rr), r = u - k * rows;
    if (y0 + r >= K2) continue;
    const double2 *line = p.buf + (r >> 1) * g.zs;
    const double2 z = line[p.pos[k]], m = line[p.pos[k == 0 ? 0 : K3 - k]];
    out[static_cast<int64_t>(k) * K1 * K2 + r] = (r & 1) ? make_double2(0.5 * (z.y + m.y), 0.5 * (m.x - z.x))
                                                         : make_double2(0.5 * (z.x + m.x), 0.5 * (z.y - m.y));
  }
}

// The inverse of k_pme_rows_fwd: phi of the rows, each led by copies of its last kPhiPad
// values.
template <typename PB>
__global__ void __launch_bounds__(kPlaneBlock) k_pme_rows_inv(const double2 *__restrict__ specs, PB pb, PmeGrid g,
                                                              double *__restrict__ phis) {
  extern __shared__ __align__(16) double plane[];
  int b, x, y0;
  rows_of(pb, g, &b, &x, &y0);
  const int K1 = pb.K[0], K2 = pb.K[1], K3 = pb.K[2], rows = 2 * g.pairs;
  const RowsLds p(plane, g);
  const int t = static_cast<int>(threadIdx.x), threads = static_cast<int>(blockDim.x);
  p.tables(g);
  __syncthreads();
  // Z_k = A_k + i B_k and Z_-k = conj(A_k) + i conj(B_k) (rows past the plane: zero)
  const double2 *in = specs + static_cast<int64_t>(pb.first + b) * g.H * K1 * K2 + static_cast<int64_t>(x) * K2 + y0;
  const float rp = __builtin_amdgcn_rcpf(static_cast<float>(g.pairs));
  for (int u = t; u < g.pairs * g.H; u += threads) {
    const int k = small_div(u, rp), j = u - k * g.pairs;
    const double2 *row = in + static_cast<int64_t>(k) * K1 * K2 + 2 * j;
    const double2 a = y0 + 2 * j < K2 ? row[0] : make_double2(0.0, 0.0);
    const double2 c = y0 + 2 * j + 1 < K2 ? row[1] : make_double2(0.0, 0.0);
    double2 *line = p.buf + j * g.zs;
    // (k = 0 and K3/2 are their own mirrors and real for both rows)
    if (k != 0 && 2 * k != K3) {
      line[p.pos[K3 - k]] = make_double2(a.x + c.y, c.x - a.y);
      line[p.pos[k]] = make_double2(a.x - c.y, a.y + c.x);
    } else {
      line[p.pos[k]] = make_double2(a.x, c.x);
    }
  }
  __syncthreads();
  fft_lines<true>([&](int l) { return [q = p.buf + l * g.zs](int e) { return q + e; }; }, g.pairs, g.f[2], p.tw);
  const int pitch = K3 + kPhiPad;
  double *out = phis + ((static_cast<int64_t>(pb.first + b) * K1 + x) * K2 + y0) * pitch;
  const int live = K2 - y0 < rows ? K2 - y0 : rows;
  const float rc = __builtin_amdgcn_rcpf(static_cast<float>(pitch));
  for (int u = t; u < live * pitch; u += threads) {
    const int r = small_div(u, rc), c = u - r * pitch;
    const int z = c < kPhiPad ? K3 - kPhiPad + c : c - kPhiPad;
    out[u] = plane[2 * ((r >> 1) * g.zs + z) + (r & 1)];
  }
}

// The (x, y) plane of one z frequency: FFTs along y and x, convolution, inverse FFTs.  One
// system has few planes (33 at 64^3), so a workgroup's own passes set its time: their LDS
// traffic (23 accesses per radix-8 butterfly, 16 without twiddles) and FP64 arithmetic on
// one CU.  C(m) is separable but for 1/m^2: exp(-pi^2 m^2/beta^2) and |b|^2 are products of
// one factor per dimension, formed once per line.
template <typename PB>
__global__ void __launch_bounds__(kPlaneBlock) k_pme_slab(double2 *__restrict__ specs, PB pb, PmeGrid g, int want,
                                                          double *__restrict__ partials_all) {
  extern __shared__ __align__(16) double plane[];
  __shared__ double red[kPlaneBlock / 64][8];
  const int b = static_cast<int>(blockIdx.x) / g.H, iz = static_cast<int>(blockIdx.x) - b * g.H;
  const int K1 = pb.K[0], K2 = pb.K[1], K3 = pb.K[2];
  double2 *buf = reinterpret_cast<double2 *>(plane);  // [K1][ys]
  double2 *tw1 = buf + K1 * g.ys, *tw2 = tw1 + K1;
  double2 *fx = tw2 + K2, *fy = fx + K1;  // by position: (factor of C, signed wave number m)
  double2 *spec = specs + (static_cast<int64_t>(pb.first + b) * g.H + iz) * K1 * K2;
  const int t = static_cast<int>(threadIdx.x), threads = static_cast<int>(blockDim.x);
  const float ry = __builtin_amdgcn_rcpf(static_cast<float>(K2));
  const int pad = g.ys - K2;
#pragma unroll 4
  for (int u = t; u < K1 * K2; u += threads) buf[u + small_div(u, ry) * pad] = spec[u];
  const PmeSys ps = make_sys(pb, b);
  for (int k = t; k < K1 + K2; k += threads) {
    const int d = k < K1 ? 0 : 1, e = d ? k - K1 : k, f = g.at[d][e];
    const double m = signed_index(f, ps.K[d]) * ps.invL[d];
    (d ? tw2 : tw1)[e] = g.tw[d][e];
    (d ? fy : fx)[e] = make_double2(g.bm[d][f] * exp(-ps.a * m * m), m);
  }
  const double mz = signed_index(iz, K3) * ps.invL[2];
  const double fz = g.bm[2][iz] * exp(-ps.a * mz * mz);
  __syncthreads();
  auto along_y = [&](int l) { return [q = buf + l * g.ys](int e) { return q + e; }; };
  auto along_x = [&](int l) { return [q = buf + l, ys = g.ys](int e) { return q + e * ys; }; };
  fft_lines<false>(along_y, K1, g.f[1], tw2);
  fft_lines<false>(along_x, K2, g.f[0], tw1);
  double v[kSymSums] = {0, 0, 0, 0, 0, 0, 0};
  const bool pair = !(iz == 0 || 2 * iz == K3);
  // the wave number of a Nyquist index (none for odd sizes)
  const double none = __builtin_inf();
  const double nyx = (K1 & 1) ? none : (K1 / 2) * ps.invL[0], nyy = (K2 & 1) ? none : (K2 / 2) * ps.invL[1];
  for (int u = t; u < K1 * K2; u += threads) {
    const int x = small_div(u, ry), y = u - x * K2;
    const double2 cx = fx[x], cy = fy[y];
    const double m[3] = {cx.y, cy.y, mz};
    const double m2 = m[0] * m[0] + m[1] * m[1] + m[2] * m[2];
    const double inv_m2 = m2 > 0.0 ? 1.0 / m2 : 0.0;  // (m = 0 is left out)
    const double C = cx.x * cy.x * fz * inv_m2, sc = 2.0 * ps.escale * C;  // sc: k_e/(pi V) C
    double2 &F = buf[u + x * pad];
    const double2 f = F;
    if (want)
      add_spec_terms(ps.escale * C * (f.x * f.x + f.y * f.y), m, 2.0 * (1.0 + ps.a * m2) * inv_m2, pair, m[0] == nyx,
                     m[1] == nyy, v);
    F = make_double2(f.x * sc, f.y * sc);
  }
  __syncthreads();
  fft_lines<true>(along_x, K2, g.f[0], tw1);
  fft_lines<true>(along_y, K1, g.f[1], tw2);
#pragma unroll 4
  for (int u = t; u < K1 * K2; u += threads) spec[u] = buf[u + small_div(u, ry) * pad];
  if (want)
    store_partials(v, red, partials_all + static_cast<int64_t>(pb.first + b) * kSymSums * g.H, g.H, iz);
}

// Sum over each aligned group of 8 lanes, in every lane (DPP moves: no LDS).
__device__ inline double octet_sum(double v) {
  auto moved = [](double x, auto ctrl) {
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(b), decltype(ctrl)::value, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(b >> 32), decltype(ctrl)::value, 0xF, 0xF, false);
    return __longlong_as_double(
        static_cast<long long>((static_cast<unsigned long long>(static_cast<unsigned>(hi)) << 32) | static_cast<unsigned>(lo)));
  };
  v += moved(v, std::integral_constant<int, 0xB1>{});   // quad_perm [1, 0, 3, 2]
  v += moved(v, std::integral_constant<int, 0x4E>{});   // quad_perm [2, 3, 0, 1]
  v += moved(v, std::integral_constant<int, 0x141>{});  // row_half_mirror
  return v;
}

// 8 lanes per atom: lane 2 a + h reads half h (two z values) of the four rows of x-plane a of
// its footprint.  Bound by the cache lines that these reads touch: two lanes share a row's
// 32 bytes.  PADDED: every row of phi starts with copies of its last three values, so that
// an atom's four z values are contiguous wherever it is; otherwise (hipFFT's grid) they are
// read one by one.  The atoms are dealt to the XCDs in contiguous ranges (workgroups go to
// the XCDs round robin), so that an XCD's L2 holds few systems' grids, or few planes.
// Workgroups past the launch's atoms each reduce one system's partials.
constexpr int kGatherLanes = 8;

template <typename T, bool PADDED, typename PB>
__global__ void __launch_bounds__(kBlock) k_pme_gather(const T *__restrict__ pos_all, const T *__restrict__ charge_all,
                                                       PB pb, const double *__restrict__ phis,
                                                       double *__restrict__ force_all,
                                                       const double *__restrict__ partials, int64_t n_part_blocks,
                                                       double *energy, double *virial) {
  __shared__ double red[kWaves][8];
  const int atom_wgs = gather_wgs(pb);
  if (static_cast<int>(blockIdx.x) >= atom_wgs) {  // workgroup-uniform
    const int64_t b = pb.first + static_cast<int>(blockIdx.x) - atom_wgs;
    reduce_sym_partials(partials + b * kSymSums * n_part_blocks, n_part_blocks, 0, n_part_blocks,
                        energy ? energy + b : nullptr, virial ? virial + 9 * b : nullptr, red);
    return;
  }
  // workgroup k of XCD x takes the k-th of range x of the atoms' workgroups
  const int xcd = static_cast<int>(blockIdx.x) % kXcds, nth = static_cast<int>(blockIdx.x) / kXcds;
  const int per = atom_wgs / kXcds, more = atom_wgs % kXcds;
  const int wg = gather_wg0(pb) + xcd * per + (xcd < more ? xcd : more) + nth;
  const int sb = system_of_wg(pb, pb.blk0, wg);
  const PmeSys ps = make_sys(pb, sb);
  const T *__restrict__ pos = pos_all + 3 * pb.a0[sb];
  const T *__restrict__ charge = charge_all + pb.a0[sb];
  const int n = pb.n[sb];
  const int pitch = PADDED ? ps.K[2] + kPhiPad : ps.K[2];
  const double *__restrict__ phi = phis + static_cast<int64_t>(pb.first + sb) * ps.K[0] * ps.K[1] * pitch;
  double *__restrict__ force = force_all + 3 * pb.a0[sb];
  const int64_t t = (static_cast<int64_t>(wg) - pb.blk0[sb]) * kBlock + threadIdx.x;
  const int i_raw = static_cast<int>(t / kGatherLanes);
  const bool valid = i_raw < n;
  const int i = valid ? i_raw : n - 1;  // lanes past the end still join the sums
  const int h = static_cast<int>(t) & 1, a = (static_cast<int>(t) >> 1) & 3;
  int ix[4], iy[4], iz[4];
  double wx[4], wy[4], wz[4], dx[4], dy[4], dz[4];
  spline4(static_cast<double>(pos[3 * static_cast<int64_t>(i) + 0]), ps.invL[0], ps.K[0], ix, wx, dx);
  spline4(static_cast<double>(pos[3 * static_cast<int64_t>(i) + 1]), ps.invL[1], ps.K[1], iy, wy, dy);
  spline4(static_cast<double>(pos[3 * static_cast<int64_t>(i) + 2]), ps.invL[2], ps.K[2], iz, wz, dz);
  auto pick = [a](const auto (&v)[4]) { return a == 0 ? v[0] : a == 1 ? v[1] : a == 2 ? v[2] : v[3]; };
  const double wxa = pick(wx), dxa = pick(dx), q = static_cast<double>(charge[i]);
  // this lane's z points: c0 = 3 - 2 h and c0 - 1 (base - c, in increasing z)
  const double w0 = h ? wz[1] : wz[3], w1 = h ? wz[0] : wz[2], d0 = h ? dz[1] : dz[3], d1 = h ? dz[0] : dz[2];
  const double *plane = phi + static_cast<int64_t>(pick(ix)) * ps.K[1] * pitch;
  const int z0 = PADDED ? iz[0] + 2 * h : (h ? iz[1] : iz[3]);  // padded: base - 3 sits at row[base]
  const int z1 = PADDED ? z0 + 1 : (h ? iz[0] : iz[2]);
  double p0[4], p1[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const double *row = plane + static_cast<int64_t>(iy[b]) * pitch;
    p0[b] = row[z0];
    p1[b] = row[z1];
  }
  double gx = 0.0, gy = 0.0, gz = 0.0;
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const double sz = p0[b] * w0 + p1[b] * w1, sdz = p0[b] * d0 + p1[b] * d1;
    gx += wy[b] * sz;
    gy += dy[b] * sz;
    gz += wy[b] * sdz;
  }
  gx = octet_sum(gx * dxa);
  gy = octet_sum(gy * wxa);
  gz = octet_sum(gz * wxa);
  if (valid && h == 0 && a < 3) {
    const double g = a == 0 ? gx : a == 1 ? gy : gz;
    const double L = a == 0 ? ps.L[0] : a == 1 ? ps.L[1] : ps.L[2];
    const int K = a == 0 ? ps.K[0] : a == 1 ? ps.K[1] : ps.K[2];
    force[3 * static_cast<int64_t>(i) + a] = -q * g * (K / L);
  }
}

// FFT plans, one forward (D2Z) and one inverse (Z2D) per grid shape, batch size and
// device, each transforming the B systems' grids (contiguous, one after the other) in
// one call; made on first use and kept for the life of the process (at most
// kMaxFftPlans of them).  The plans do not allocate their work buffers: every call hands
// them the work area of its own workspace, so calls on different streams with different
// workspaces share nothing but the plans' read-only tables.  The mutex covers the cache
// and, per call, setting a plan's stream and work area and enqueueing its transform.
struct FftPlans {
  hipfftHandle fwd = nullptr, inv = nullptr;
  size_t work = 0;  // bytes of work area either transform needs
};
constexpr size_t kMaxFftPlans = 32;
std::mutex g_fft_mu;
std::map<std::tuple<int, int, int, int, int>, FftPlans> g_fft;

const char *fft_error(hipfftResult r) {
  switch (r) {
    case HIPFFT_ALLOC_FAILED: return "FFT allocation failed";
    case HIPFFT_INVALID_SIZE: return "FFT size refused";
    case HIPFFT_EXEC_FAILED: return "FFT execution failed";
    default: return "FFT library error";
  }
}

// The plans for this layout on the current device, made if needed.  Returns "" or the
// reason they could not be made.  Caller holds g_fft_mu.
std::string fft_plans_locked(int B, const int K[3], int64_t grid, int64_t spec, FftPlans *out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return "no current HIP device";
  const auto key = std::make_tuple(dev, K[0], K[1], K[2], B);
  auto it = g_fft.find(key);
  if (it != g_fft.end()) {
    *out = it->second;
    return "";
  }
  if (g_fft.size() >= kMaxFftPlans)
    return "more than 32 distinct (grid shape, batch size, device) FFT plans in this process";
  FftPlans p;
  int dims[3] = {K[0], K[1], K[2]};
  // contiguous grids, unit stride: K1 K2 K3 reals and K1 K2 (K3/2+1) complex values per
  // system, one system after the other
  int real_embed[3] = {K[0], K[1], K[2]};
  int spec_embed[3] = {K[0], K[1], K[2] / 2 + 1};
  const int grid_dist = static_cast<int>(grid), spec_dist = static_cast<int>(spec);
  size_t wf = 0, wi = 0;
  hipfftResult r = hipfftCreate(&p.fwd);
  if (r == HIPFFT_SUCCESS) r = hipfftSetAutoAllocation(p.fwd, 0);
  if (r == HIPFFT_SUCCESS)
    r = hipfftMakePlanMany(p.fwd, 3, dims, real_embed, 1, grid_dist, spec_embed, 1, spec_dist, HIPFFT_D2Z, B, &wf);
  if (r != HIPFFT_SUCCESS) {
    if (p.fwd) hipfftDestroy(p.fwd);
    return std::string("hipfftMakePlanMany (D2Z): ") + fft_error(r);
  }
  r = hipfftCreate(&p.inv);
  if (r == HIPFFT_SUCCESS) r = hipfftSetAutoAllocation(p.inv, 0);
  if (r == HIPFFT_SUCCESS)
    r = hipfftMakePlanMany(p.inv, 3, dims, spec_embed, 1, spec_dist, real_embed, 1, grid_dist, HIPFFT_Z2D, B, &wi);
  if (r != HIPFFT_SUCCESS) {
    hipfftDestroy(p.fwd);
    if (p.inv) hipfftDestroy(p.inv);
    return std::string("hipfftMakePlanMany (Z2D): ") + fft_error(r);
  }
  p.work = std::max(wf, wi);
  g_fft.emplace(key, p);
  *out = p;
  return "";
}

}  // namespace

namespace {
// Shapes of a grid transformed here, for a batch of B systems (table pointers apart); false
// when it goes through hipFFT (a prime factor above 7, or rows or a slab too large for LDS).
bool pme_grid(const int K[3], int B, PmeGrid *out) {
  PmeGrid g{};
  for (int a = 0; a < 3; ++a)
    if (!fft_shape(K[a], &g.f[a])) return false;
  g.H = K[2] / 2 + 1;
  g.zs = K[2] | 1;
  g.ys = K[1] | 1;
  // workgroups per x-plane: enough to have one on each of the 256 CUs, at most 4 (each
  // looks at all of the plane's atoms)
  const int want = std::min<int64_t>(4, (kCus + static_cast<int64_t>(K[0]) * B - 1) / (static_cast<int64_t>(K[0]) * B));
  const int all = (K[1] + 1) / 2;  // row pairs of a plane
  g.pairs = (all + want - 1) / want;
  g.blocks = (all + g.pairs - 1) / g.pairs;
  while (rows_lds_bytes(g) > kPmeLdsMax && g.pairs > 1) {
    g.pairs = (g.pairs + 1) / 2;
    g.blocks = (all + g.pairs - 1) / g.pairs;
  }
  if (rows_lds_bytes(g) > kPmeLdsMax || slab_lds_bytes(g) > kPmeLdsMax) return false;
  *out = g;
  return true;
}

constexpr size_t kTableBytes = 2 * 24 + 8 + 3 * 4;  // of a PmeTable, per system

int64_t bin_workgroups(const nb_system *sys, int b) {
  return std::max<int64_t>(sys->atom_offset[b + 1] - sys->atom_offset[b] + kBinAtoms - 1, 0) / kBinAtoms;
}
}  // namespace

std::string pme_layout(int B, const int32_t grid[3], PmeLayout *lay) {
  if (!grid) return "grid is NULL";
  for (int a = 0; a < 3; ++a)
    if (grid[a] < kMinGrid || grid[a] > kMaxGrid) return "grid sizes must be in [4, 1024]";
  PmeLayout l;
  l.B = B;
  for (int a = 0; a < 3; ++a) l.K[a] = grid[a];
  l.grid = static_cast<int64_t>(grid[0]) * grid[1] * grid[2];
  l.spec = static_cast<int64_t>(grid[0]) * grid[1] * (grid[2] / 2 + 1);
  if (l.grid > (int64_t{1} << 28)) return "grid larger than 2^28 points";
  if (static_cast<int64_t>(B) * l.grid > (int64_t{1} << 31)) return "batch grids larger than 2^31 points";
  l.conv_blocks = (l.spec + kBlock - 1) / kBlock;
  PmeGrid g;
  l.in_lds = pme_grid(l.K, B, &g);
  size_t off = 0, real_bytes = sizeof(double) * static_cast<size_t>(B) * l.grid;
  // (the padded potential, in whose place the binned atoms wait until the planes are summed)
  if (l.in_lds) real_bytes += sizeof(double) * kPhiPad * static_cast<size_t>(B) * grid[0] * grid[1];
  l.real = off;
  off = align256(off + real_bytes);
  l.cplx = off;
  off = align256(off + 2 * sizeof(double) * static_cast<size_t>(B) * l.spec);
  l.partials = off;
  off = align256(off + sizeof(double) * static_cast<size_t>(B) * kPart * std::max<int64_t>(l.conv_blocks, l.K[2] / 2 + 1));
  l.tables = off;
  if (l.in_lds) off = align256(off + (16 + 8 + 4) * static_cast<size_t>(l.K[0] + l.K[1] + l.K[2]));
  l.systems = off;
  if (l.in_lds && B > kPmeChunk) off = align256(off + kTableBytes * (static_cast<size_t>(B) + 1));
  l.work = off;
  l.total = off;
  *lay = l;
  return "";
}

std::string pme_attach_plans(PmeLayout *lay) {
  if (lay->in_lds) return "";  // no FFT library plans
  FftPlans plans;
  {
    std::lock_guard<std::mutex> lock(g_fft_mu);
    const std::string why = fft_plans_locked(lay->B, lay->K, lay->grid, lay->spec, &plans);
    if (!why.empty()) return why;
  }
  lay->work_bytes = plans.work;
  lay->total = align256(lay->work + plans.work);
  return "";
}

namespace {

// The launch descriptor of systems [first, first + nsys).  bins: the binning workgroups of the
// systems before them, to be carried on (null: the atoms are not binned); before: likewise the
// gather's (null: counted from these systems on).
template <int CAP>
PmeBatch<CAP> pme_chunk(const PmeLayout &lay, const nb_system *sys, double a, double ke, int first, int nsys,
                        int32_t *bins, int32_t *before = nullptr) {
  PmeBatch<CAP> pb;
  std::memset(&pb, 0, sizeof(pb));
  pb.nsys = nsys;
  pb.first = first;
  for (int d = 0; d < 3; ++d) pb.K[d] = lay.K[d];
  pb.a = a;
  pb.ke = ke;
  int32_t blocks = before ? *before : 0;
  for (int k = 0; k < nsys; ++k) {
    const int b = first + k;
    for (int d = 0; d < 3; ++d) {
      pb.L[k][d] = sys->box[3 * b + d];
      pb.invL[k][d] = 1.0 / pb.L[k][d];
    }
    pb.a0[k] = sys->atom_offset[b];
    pb.n[k] = static_cast<int32_t>(sys->atom_offset[b + 1] - sys->atom_offset[b]);
    pb.blk0[k] = blocks;
    blocks += static_cast<int32_t>((static_cast<int64_t>(pb.n[k]) * kGatherLanes + kBlock - 1) / kBlock);
    if (!bins) continue;
    pb.bin0[k] = *bins;
    *bins += static_cast<int32_t>(bin_workgroups(sys, b));
  }
  pb.blk0[nsys] = blocks;
  if (bins) pb.bin0[nsys] = *bins;
  if (before) *before = blocks;
  return pb;
}

template <int CAP>
int32_t gather_wgs_host(const PmeBatch<CAP> &pb) { return pb.blk0[pb.nsys]; }
int32_t gather_wgs_host(const PmeTable &pb) { return pb.wgs; }

template <bool PADDED, typename PB>
void launch_gather(const PB &pb, const nb_system *sys, const double *phi, double *force, const double *partials,
                   int64_t n_part_blocks, double *energy, double *virial, hipStream_t s) {
  const unsigned grid = static_cast<unsigned>(gather_wgs_host(pb) + ((energy || virial) ? pb.nsys : 0));
  if (grid == 0) return;
  if (sys->pos_is_f64)
    hipLaunchKernelGGL((k_pme_gather<double, PADDED, PB>), dim3(grid), dim3(kBlock), 0, s,
                       static_cast<const double *>(sys->pos), static_cast<const double *>(sys->charge), pb, phi, force,
                       partials, n_part_blocks, energy, virial);
  else
    hipLaunchKernelGGL((k_pme_gather<float, PADDED, PB>), dim3(grid), dim3(kBlock), 0, s,
                       static_cast<const float *>(sys->pos), static_cast<const float *>(sys->charge), pb, phi, force,
                       partials, n_part_blocks, energy, virial);
}

// A grid transformed in LDS: five launches.  CAP: systems that travel in one launch's arguments;
// a larger batch bins CAP at a time, and the other launches find its systems in the table.
template <int CAP>
hipError_t launch_pme_lds(const PmeLayout &lay, const nb_system *sys, double beta, double ke, char *base,
                          double *force, double *energy, double *virial, hipStream_t s) {
  PmeGrid g;
  if (!pme_grid(lay.K, lay.B, &g)) return hipErrorInvalidValue;
  double *phi = reinterpret_cast<double *>(base + lay.real);
  // The atoms are binned where they fit into the potential's place (32 bytes each against 8 a
  // grid point: grids of more than four points per atom, twice as coarse as one point per
  // Angstrom, or finer).  Otherwise the rows kernel reads all of a system's atoms for each of its
  // planes, so that the workspace depends on the number of systems and the grid alone.
  const size_t atom_bytes = align256(sizeof(PmeAtom) * static_cast<size_t>(sys->atom_offset[lay.B]));
  size_t bin_wgs = 0;
  for (int b = 0; b < lay.B; ++b) bin_wgs += static_cast<size_t>(bin_workgroups(sys, b));
  const bool binned = atom_bytes + sizeof(uint16_t) * bin_wgs * (lay.K[0] + 1) <= lay.cplx - lay.real;
  PmeAtom *atoms = reinterpret_cast<PmeAtom *>(base + lay.real);
  uint16_t *offs = reinterpret_cast<uint16_t *>(base + lay.real + atom_bytes);
  double2 *spec = reinterpret_cast<double2 *>(base + lay.cplx);
  double *partials = reinterpret_cast<double *>(base + lay.partials);
  char *tab = base + lay.tables;
  const int sum_k = lay.K[0] + lay.K[1] + lay.K[2];
  for (int d = 0, k = 0; d < 3; k += lay.K[d++]) {
    g.tw[d] = reinterpret_cast<double2 *>(tab) + k;
    g.bm[d] = reinterpret_cast<double *>(tab + 16 * static_cast<size_t>(sum_k)) + k;
    g.at[d] = reinterpret_cast<int32_t *>(tab + 24 * static_cast<size_t>(sum_k)) + k;
  }
  const double a = kPi * kPi / (beta * beta);
  const int want = (energy || virial) ? 1 : 0;
  const size_t rows_lds = rows_lds_bytes(g), slab_lds = slab_lds_bytes(g);
  // Threads per workgroup: as many as shorten one workgroup's passes while the grid does not
  // fill the chip, 256 (more workgroups per CU, whose phases overlap) when it does.  A slab of
  // 1,024 threads has a CU to itself by its registers: from 257 on they would queue, so 512 and
  // then 256, but for planes that have it by their LDS in any case (call, 1,024 against 512
  // threads: 264 slabs of 20 x 20 46 and 38 us, 264 of 64 x 64 96 and 86; 276 of 90 x 90 177
  // and 184).
  const int rows_wgs = lay.K[0] * g.blocks * lay.B, slab_wgs = g.H * lay.B;
  const bool alone = slab_wgs <= kCus || 2 * slab_lds > kPmeLdsMax;
  const dim3 rows_thr(rows_wgs > 2 * kCus ? 256 : 512);
  const dim3 slab_thr(alone ? kPlaneBlock : slab_wgs > 2 * kCus ? 256 : 512);
  const bool f64 = sys->pos_is_f64 != 0;
  const auto *pos64 = static_cast<const double *>(sys->pos), *q64 = static_cast<const double *>(sys->charge);
  const auto *pos32 = static_cast<const float *>(sys->pos), *q32 = static_cast<const float *>(sys->charge);
  // The steps after the binning, each for all of the batch before the next (phi takes the bins'
  // place), in launches of the systems of each of parts.
  auto steps = [&](const auto &parts) {
    using PB = std::remove_cv_t<std::remove_reference_t<decltype(*std::begin(parts))>>;
    auto row_wgs = [&](const PB &pb) { return dim3(static_cast<unsigned>(lay.K[0] * g.blocks * pb.nsys)); };
    auto rows = [&](const PB &pb, const auto *from, const auto *beside) {
      using T = std::remove_const_t<std::remove_reference_t<decltype(*from)>>;
      using U = std::remove_const_t<std::remove_reference_t<decltype(*beside)>>;
      hipLaunchKernelGGL((k_pme_rows_fwd<T, U, PB>), row_wgs(pb), rows_thr, rows_lds, s, from, beside, pb, g, spec);
    };
    for (const PB &pb : parts) {
      if (binned) rows(pb, atoms, offs);
      else if (f64) rows(pb, pos64, q64);
      else rows(pb, pos32, q32);
    }
    for (const PB &pb : parts)
      hipLaunchKernelGGL(k_pme_slab<PB>, dim3(static_cast<unsigned>(g.H * pb.nsys)), slab_thr, slab_lds, s, spec, pb, g,
                         want, partials);
    for (const PB &pb : parts)
      hipLaunchKernelGGL(k_pme_rows_inv<PB>, row_wgs(pb), rows_thr, rows_lds, s, spec, pb, g, phi);
    for (const PB &pb : parts) launch_gather<true>(pb, sys, phi, force, partials, g.H, energy, virial, s);
  };
  int32_t bins = 0, *const binning = binned ? &bins : nullptr;
  if (lay.B <= CAP) {
    const PmeBatch<CAP> all[1] = {pme_chunk<CAP>(lay, sys, a, ke, 0, lay.B, binning)};
    const PmeBatch<CAP> &pb = all[0];
    const dim3 wgs(static_cast<unsigned>(bins) + 3u);
    if (f64) hipLaunchKernelGGL((k_pme_bin<double, CAP>), wgs, dim3(kBinAtoms), 0, s, pos64, q64, pb, g, atoms, offs);
    else hipLaunchKernelGGL((k_pme_bin<float, CAP>), wgs, dim3(kBinAtoms), 0, s, pos32, q32, pb, g, atoms, offs);
    steps(all);
    return hipGetLastError();
  }
  if constexpr (CAP == kPmeChunk) {
    const size_t B = static_cast<size_t>(lay.B);
    char *at = base + lay.systems;
    PmeTable tab{};
    tab.L = reinterpret_cast<double(*)[3]>(at);
    tab.invL = tab.L + B;
    tab.a0 = reinterpret_cast<int64_t *>(tab.invL + B);
    tab.n = reinterpret_cast<int32_t *>(tab.a0 + B);
    tab.blk0 = tab.n + B;
    tab.bin0 = tab.blk0 + B + 1;
    for (int d = 0; d < 3; ++d) tab.K[d] = lay.K[d];
    tab.a = a;
    tab.ke = ke;
    // (a launch has fewer than 2^32 threads: ranges of at most 2^20 workgroups, or one system)
    const int64_t most = std::max<int64_t>(static_cast<int64_t>(lay.K[0]) * g.blocks, g.H);
    static_assert(kBlock / kGatherLanes == 32, "atoms per gather workgroup");
    auto gather_wgs = [&](int b) { return (sys->atom_offset[b + 1] - sys->atom_offset[b] + 31) / 32; };
    std::vector<PmeTable> parts;
    for (int first = 0, end; first < lay.B; first = end) {
      int64_t wgs = gather_wgs(first);
      for (end = first + 1; end < lay.B; ++end) {
        const int64_t more = gather_wgs(end);
        if (wgs + more > (1 << 20) || (end + 1 - first) * most > (1 << 20)) break;
        wgs += more;
      }
      PmeTable part = tab;
      part.first = first;
      part.nsys = end - first;
      part.wgs = static_cast<int>(wgs);
      part.L += first, part.invL += first, part.a0 += first, part.n += first, part.blk0 += first, part.bin0 += first;
      parts.push_back(part);
      tab.wg0 += part.wgs;
    }
    int32_t gathers = 0;
    for (int first = 0; first < lay.B; first += CAP) {
      const PmeBatch<CAP> pb = pme_chunk<CAP>(lay, sys, a, ke, first, std::min(CAP, lay.B - first), binning, &gathers);
      const dim3 wgs(static_cast<unsigned>(pb.bin0[pb.nsys] - pb.bin0[0]) + (first == 0 ? 3u : 0u) + 1u);
      if (f64)
        hipLaunchKernelGGL(k_pme_bin_table<double>, wgs, dim3(kBinAtoms), 0, s, pos64, q64, pb, g, atoms, offs, tab);
      else hipLaunchKernelGGL(k_pme_bin_table<float>, wgs, dim3(kBinAtoms), 0, s, pos32, q32, pb, g, atoms, offs, tab);
    }
    steps(parts);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_pme(const PmeLayout &lay, const nb_system *sys, double beta, double ke, void *ws, double *force,
                      double *energy, double *virial, hipStream_t s, std::string *err) {
  char *base = static_cast<char *>(ws);
  if (lay.in_lds)
    return lay.B == 1 ? launch_pme_lds<1>(lay, sys, beta, ke, base, force, energy, virial, s)
                      : launch_pme_lds<kPmeChunk>(lay, sys, beta, ke, base, force, energy, virial, s);
  double *real = reinterpret_cast<double *>(base + lay.real);
  double2 *cplx = reinterpret_cast<double2 *>(base + lay.cplx);
  double *partials = reinterpret_cast<double *>(base + lay.partials);
  void *work = lay.work_bytes ? static_cast<void *>(base + lay.work) : nullptr;
  auto stride_blocks = [](int64_t n) {
    return dim3(static_cast<unsigned>(std::min<int64_t>((n + kBlock - 1) / kBlock, 65536)));
  };
  FftPlans plans;
  {
    std::lock_guard<std::mutex> lock(g_fft_mu);
    const std::string why = fft_plans_locked(lay.B, lay.K, lay.grid, lay.spec, &plans);
    if (!why.empty()) {
      *err = why;
      return hipErrorUnknown;
    }
  }
  if (plans.work > lay.work_bytes) {  // the workspace was sized for another device's plans
    *err = "workspace sized for FFT plans of another device";
    return hipErrorUnknown;
  }
  const int64_t plane_points = static_cast<int64_t>(lay.K[1]) * lay.K[2];
  const bool planes = plane_points <= kPlaneMaxPoints;
  const bool f64 = sys->pos_is_f64 != 0;
  const double a = kPi * kPi / (beta * beta);
  auto chunk = [&](int first, int nsys) { return pme_chunk<kPmeChunk>(lay, sys, a, ke, first, nsys, nullptr); };
  const dim3 blk(kBlock);
  // charge grids
  if (!planes)
    hipLaunchKernelGGL(k_pme_zero, stride_blocks(lay.grid * lay.B), dim3(kBlock), 0, s, real, lay.grid * lay.B);
  for (int first = 0; first < lay.B; first += kPmeChunk) {
    const PmeBatch<kPmeChunk> pb = chunk(first, std::min(kPmeChunk, lay.B - first));
    if (planes) {
      const dim3 gp(static_cast<unsigned>(lay.K[0] * pb.nsys)), bp(kPlaneBlock);
      const size_t lds = sizeof(double) * static_cast<size_t>(plane_points);
      if (f64)
        hipLaunchKernelGGL(k_pme_spread_planes<double>, gp, bp, lds, s, static_cast<const double *>(sys->pos),
                           static_cast<const double *>(sys->charge), pb, lay.grid, real);
      else
        hipLaunchKernelGGL(k_pme_spread_planes<float>, gp, bp, lds, s, static_cast<const float *>(sys->pos),
                           static_cast<const float *>(sys->charge), pb, lay.grid, real);
    } else {
      for (int k = 0; k < pb.nsys; ++k) {  // grids too large for a plane in LDS: per system
        const int64_t n = pb.n[k];
        if (n == 0) continue;
        const PmeSys ps = make_sys(pb, k);
        double *g = real + static_cast<int64_t>(first + k) * lay.grid;
        const dim3 ga(static_cast<unsigned>((n * kLanesPerAtom + kBlock - 1) / kBlock));
        if (f64)
          hipLaunchKernelGGL(k_pme_spread<double>, ga, blk, 0, s, static_cast<const double *>(sys->pos) + 3 * pb.a0[k],
                             static_cast<const double *>(sys->charge) + pb.a0[k], static_cast<int>(n), ps, g);
        else
          hipLaunchKernelGGL(k_pme_spread<float>, ga, blk, 0, s, static_cast<const float *>(sys->pos) + 3 * pb.a0[k],
                             static_cast<const float *>(sys->charge) + pb.a0[k], static_cast<int>(n), ps, g);
      }
    }
  }
  {
    std::lock_guard<std::mutex> lock(g_fft_mu);
    hipfftResult r = hipfftSetStream(plans.fwd, s);
    if (r == HIPFFT_SUCCESS) r = hipfftSetWorkArea(plans.fwd, work);
    if (r == HIPFFT_SUCCESS) r = hipfftExecD2Z(plans.fwd, real, reinterpret_cast<hipfftDoubleComplex *>(cplx));
    if (r != HIPFFT_SUCCESS) {
      *err = std::string("hipfftExecD2Z: ") + fft_error(r);
      return hipErrorUnknown;
    }
  }
  for (int first = 0; first < lay.B; first += kPmeChunk) {  // convolution, energy and virial partials
    const PmeBatch<kPmeChunk> pb = chunk(first, std::min(kPmeChunk, lay.B - first));
    hipLaunchKernelGGL(k_pme_convolve, dim3(static_cast<unsigned>(lay.conv_blocks * pb.nsys)), blk, 0, s, cplx, pb,
                       lay.spec, partials, lay.conv_blocks);
  }
  {
    std::lock_guard<std::mutex> lock(g_fft_mu);
    hipfftResult r = hipfftSetStream(plans.inv, s);
    if (r == HIPFFT_SUCCESS) r = hipfftSetWorkArea(plans.inv, work);
    if (r == HIPFFT_SUCCESS) r = hipfftExecZ2D(plans.inv, reinterpret_cast<hipfftDoubleComplex *>(cplx), real);
    if (r != HIPFFT_SUCCESS) {
      *err = std::string("hipfftExecZ2D: ") + fft_error(r);
      return hipErrorUnknown;
    }
  }
  // forces from the potential grids, energies and virials
  for (int first = 0; first < lay.B; first += kPmeChunk)
    launch_gather<false>(chunk(first, std::min(kPmeChunk, lay.B - first)), sys, real, force, partials, lay.conv_blocks,
                         energy, virial, s);
  return hipGetLastError();
}

}  // namespace nb
