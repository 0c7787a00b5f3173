// lb_step.hip -- instantiation of the step kernels for one storage type LB_S
// and one collision operator LB_C (both given on the compiler command line).
#include <hip/hip_runtime.h>

#include "lb_kernels.hpp"
#include "lb_launch.hpp"

#if !defined(LB_S) || !defined(LB_C)
#error "compile with -DLB_S=<0|1|2> -DLB_C=<0|1|2>"
#endif

namespace lbhost {

using namespace lbdev;

template <int S, int C, bool P, int E, bool AA>
void launch_lb(dim3 g, hipStream_t s, const LbArgs& a) {
  hipLaunchKernelGGL((k_lb<S, C, P, WG, E, AA>), g, dim3(WG), 0, s, a);
}

template <int S, int C, int E>
LbLaunch pick_lb_ext(bool periodic, bool in_place) {
  if (periodic) return in_place ? launch_lb<S, C, true, E, true> : launch_lb<S, C, true, E, false>;
  return in_place ? launch_lb<S, C, false, E, true> : launch_lb<S, C, false, E, false>;
}

template <int S, int C>
LbLaunch pick_lb(bool periodic, int ext, bool in_place) {
  if constexpr (C != 0) {
    if (ext == 2) return pick_lb_ext<S, C, 2>(periodic, in_place);
  }
  return ext ? pick_lb_ext<S, C, 1>(periodic, in_place) : pick_lb_ext<S, C, 0>(periodic, in_place);
}

template LbLaunch pick_lb<LB_S, LB_C>(bool, int, bool);

template <int S, int C, bool P, int E>
void launch_force(dim3 g, hipStream_t s, const LbArgs& a) {
  hipLaunchKernelGGL((k_force<S, C, P, E>), g, dim3(WG), 0, s, a);
}

template <int S, int C>
LbLaunch pick_force(bool periodic, int ext) {
  if constexpr (C != 0) {
    if (ext == 2) return periodic ? launch_force<S, C, true, 2> : launch_force<S, C, false, 2>;
  }
  if (ext) return periodic ? launch_force<S, C, true, 1> : launch_force<S, C, false, 1>;
  return periodic ? launch_force<S, C, true, 0> : launch_force<S, C, false, 0>;
}

template LbLaunch pick_force<LB_S, LB_C>(bool, int);

#if LB_C == 0
template <int S, bool P, int MB, bool TH>
void launch_chain(int nch, hipStream_t s, const BoxDesc* boxes, const ChainDesc* chains,
                  const void* a0, const void* a1, void* pos, void* vel, int total, int4* rb,
                  void* rd, void* rp, int* bbox, double* gtab, DevState* st, double rho0, int pre,
                  long long* stamp, const int4* xf_items, int n_xf, float* xface, unsigned key0,
                  unsigned key1) {
  using T = typename Store<S>::T;
  // one workgroup per chain, then an x-face work item per wavefront
  constexpr int NT = chain_threads(MB);
  const int nxb = (n_xf + NT / 64 - 1) / (NT / 64);
  hipLaunchKernelGGL((k_chain<S, P, MB, TH>), dim3(nch + nxb), dim3(NT), 0, s, boxes, chains,
                     (const T*)a0, (const T*)a1, (double*)pos, (double*)vel, total, rb, (double*)rd,
                     (double*)rp, bbox, gtab, st, rho0, pre, stamp, nch, xf_items, n_xf, xface, key0, key1);
}

template <int S, bool TH>
ChainLaunch pick_chain_th(bool periodic, int max_beads) {
  if (max_beads <= 64) return periodic ? launch_chain<S, true, 64, TH> : launch_chain<S, false, 64, TH>;
  return periodic ? launch_chain<S, true, 256, TH> : launch_chain<S, false, 256, TH>;
}

template <int S>
ChainLaunch pick_chain(bool periodic, int max_beads, bool thermal) {
  return thermal ? pick_chain_th<S, true>(periodic, max_beads)
                 : pick_chain_th<S, false>(periodic, max_beads);
}

template ChainLaunch pick_chain<LB_S>(bool, int, bool);
#endif

}  // namespace lbhost
