// Ewald corrections around the real-space pair term (ACEMD paper, section 3: the
// electrostatics are PME, and the pair kernels compute its real-space part).  The
// reciprocal part counts every pair, excluded ones included, and every charge with
// itself; these corrections take out
//
//   for every excluded pair {i, j} (the union of both atoms' exclusion rows, at any
//   distance, minimum image):   u_ij = -k_e q_i q_j erf(beta r) / r
//                               (at r = 0 its limit -k_e q_i q_j 2 beta / sqrt(pi))
//   for every atom:             -k_e beta / sqrt(pi) q_i^2
//   for every scaled 1-4 pair {i, j} that is not excluded (the union of both 1-4 rows,
//   within the 64-index window): (1 - s14_coul) u_ij, so that with the pair kernels'
//   s14_coul erfc term and the reciprocal part the whole Coulomb interaction of the pair
//   is s14_coul k_e q_i q_j / r.
//
// The force on i from pair {i, j} is g_ij d_ij with
//   g_ij = k_e q_i q_j [(2 beta / sqrt(pi)) exp(-beta^2 r^2) / r^2 - erf(beta r) / r^3].
//
// A few pairs per atom: FP64 arithmetic on the caller's own arrays for both precisions.
// One thread per atom (caller's order) gathers its force from
//   * the partners inside its 128-bit exclusion window, from the bitmaps of the cell
//     build (which hold the union of both rows), each pair seen from both sides, and
//   * the far entries of its own row (|j - i| > 64), counted in full on this side when
//     the partner's row does not list the atom, by halves otherwise;
// a second launch adds each far pair listed in one row only to the other atom's force
// (FP64 atomics: the only additions whose order can vary, and only for atoms with more
// than one such pair), and reduces the first one's per-block energy and virial partials
// per system in a fixed order.  Both are bound by latency (one wave per SIMD on the
// 23.6k-atom box, a chain of dependent loads and one erf per partner): the partners'
// loads are issued together, and sums that nobody asked for are not formed.  With the
// far pass and the reduction in launches of their own and ten sums reduced one by one the
// GPU worked 15 us there (8.6 + 2.5 + 4.0 traced); now 9 (5.6 + 3.1), and the call, bound by
// the host, takes 10.3.
#include "nb_internal.h"
#include "nb_ewald.h"
#include "nb_pair_common.h"

namespace nb {

namespace {

template <typename T, bool WANT>
__global__ void __launch_bounds__(kBlock) k_ewald_atoms(Dev d, EwaldArgs<T> a, double *force) {
  __shared__ double red[kWaves][8];
  if (!built_for(d.status, d.N, false, false)) {
    if (blockIdx.x == 0 && threadIdx.x == 0) atomicOr(d.status, NB_STATUS_NOT_BUILT);
    return;
  }
  ewald_atoms<T, WANT>(d, a, force, static_cast<int>(blockIdx.x), red);
}

// Workgroups [0, far_wgs): the far pass; then one per system: its energy and virial, its
// blocks' partials in order.
template <typename T>
__global__ void __launch_bounds__(kBlock) k_ewald_finish(Dev d, EwaldArgs<T> a, double *force, int far_wgs,
                                                         double *energy, double *virial) {
  __shared__ double red[kWaves][8];
  if (!built_for(d.status, d.N, false, false)) return;
  if (static_cast<int>(blockIdx.x) < far_wgs) {
    ewald_far<T>(d, a, force, static_cast<int>(blockIdx.x));
    return;
  }
  const int b = static_cast<int>(blockIdx.x) - far_wgs;
  const int64_t lo = d.desc[b].blk_begin, hi = b + 1 < d.B ? d.desc[b + 1].blk_begin : d.n_blocks;
  reduce_sym_partials(d.partials, d.n_slots, lo, hi, energy ? energy + b : nullptr, virial ? virial + 9 * b : nullptr,
                      red);
}

template <typename T>
void launch_ewald_as(const Plan &p, const Dev &d, const nb_system *sys, double *force, double *energy, double *virial,
                     hipStream_t s) {
  const EwaldArgs<T> a = ewald_args<T>(p, sys);
  const bool want = energy || virial;
  const dim3 grid(static_cast<unsigned>(p.n_blocks)), block(kBlock);
  // A batch without atoms launches no per-atom work, but its systems' energies and
  // virials are still written (zeros: a system without blocks sums to nothing).
  if (p.n_blocks > 0) {
    if (want) hipLaunchKernelGGL((k_ewald_atoms<T, true>), grid, block, 0, s, d, a, force);
    else hipLaunchKernelGGL((k_ewald_atoms<T, false>), grid, block, 0, s, d, a, force);
  }
  const unsigned wgs = static_cast<unsigned>(p.n_blocks + (want ? p.B : 0));
  if (wgs > 0)
    hipLaunchKernelGGL(k_ewald_finish<T>, dim3(wgs), block, 0, s, d, a, force, static_cast<int>(p.n_blocks), energy,
                       virial);
}

}  // namespace

hipError_t launch_ewald(const Plan &p, const Dev &d, const nb_system *sys, double *force, double *energy,
                        double *virial, hipStream_t s) {
  if (sys->pos_is_f64) launch_ewald_as<double>(p, d, sys, force, energy, virial, s);
  else launch_ewald_as<float>(p, d, sys, force, energy, virial, s);
  return hipGetLastError();
}

}  // namespace nb
