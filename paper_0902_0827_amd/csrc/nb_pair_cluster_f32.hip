// Mixed-precision (FP32 pair arithmetic) instantiations of the cluster pair kernel for
// forces, and the finishing pass shared by both precisions.
#include "nb_pair_cluster.h"

namespace nb {

void launch_cluster_forces_f64(const Plan &p, const Dev &d, const Consts &c, const Out &o, bool half, hipStream_t s);
void launch_cluster_grad_f32(const Plan &p, const Dev &d, const Consts &c, const Out &o, int mode, bool half,
                             hipStream_t s);
void launch_cluster_grad_f64(const Plan &p, const Dev &d, const Consts &c, const Out &o, int mode, bool half,
                             hipStream_t s);

void launch_cluster_pair(const Plan &p, const Dev &whole, const Consts &c, const Out &o, int mode, hipStream_t s,
                         double *energy, double *virial, const double *eps, double *grad_sigma, double *grad_eps) {
  const Dev d = parts_view(p, whole, mode);
  // the adjoint and the force VJP stay full-shell
  const bool half = p.kernel == NB_KERNEL_CLUSTER_HALF && mode != kAdjoint && mode != kVJP;
  const bool f64 = p.precision == NB_FP64;
  if (mode != kForces) (f64 ? launch_cluster_grad_f64 : launch_cluster_grad_f32)(p, d, c, o, mode, half, s);
  else if (f64) launch_cluster_forces_f64(p, d, c, o, half, s);
  else launch_cluster_pair_prec<false, false>(p, d, c, o, mode, half, s);
  if (o.skip_finish) return;
  // With one item per cluster the full-shell kernel has written the per-atom outputs
  // itself; the half-shell kernel's accumulators are always copied out here.
  const int parts = p.split * pair_parts(p, mode);  // of every cluster's candidates
  const int blocksA = static_cast<int>((p.N + kFinishBlock - 1) / kFinishBlock);
  const int nA = half ? ((mode == kForces || o.atom_energy) ? blocksA : 0) : (parts == 1 ? 0 : blocksA);
  int nv = 0;
  if (mode == kForces) nv = o.want_part ? (virial ? kPart : 1) : 0;
  if (mode == kEnergy) nv = 1;
  const int extra = (mode == kAdjoint || mode == kVJP) ? ((grad_sigma || grad_eps) ? 2 * p.T : 0) : 0;
  const dim3 fg(static_cast<unsigned>(nA + kPart * p.B + extra));
  const uint32_t key = cluster_key(p);
  auto finish = [&](auto mode_c, int is_half) {
    constexpr int MODE = decltype(mode_c)::value;
    auto *kern = long_sums(p, parts) ? k_finish<MODE, true> : k_finish<MODE, false>;
    hipLaunchKernelGGL(kern, fg, dim3(kFinishBlock), 0, s, d, o, parts, nA, energy, virial, nv, eps, grad_sigma,
                       grad_eps, is_half, key);
  };
  if (mode == kForces) finish(std::integral_constant<int, kForces>{}, half ? 1 : 0);
  else if (mode == kEnergy) finish(std::integral_constant<int, kEnergy>{}, half ? 1 : 0);
  else if (mode == kVJP) finish(std::integral_constant<int, kVJP>{}, 0);
  else finish(std::integral_constant<int, kAdjoint>{}, 0);
}

}  // namespace nb
