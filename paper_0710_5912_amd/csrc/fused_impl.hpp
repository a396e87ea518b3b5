// fused_impl.hpp -- launchers of the four-pass row kernels (included once per
// precision by fused_f64.hip / fused_f32.hip).
#pragma once

#include "fused.hpp"

namespace le {

template <typename T, int L>
struct FusedLaunch {
  static constexpr int EW = L >= 1024 ? 16 : (L >= 8 ? 8 : L);  // the wide shapes
  static constexpr int EN = L >= 4 && L <= 256 ? 4 : EW;
  template <int NR, int NF, int E>
  static bool adv(const Run* runs, int nruns, int ny, const StepArgs* sa, hipStream_t st) {
    using C = FuseCfg<T, L, NR, NF, E>;
    if constexpr (C::AOK) {
      if (nruns > 0)
          hipLaunchKernelGGL((k_flow_adv<T, 2 * L, NR, NF, E>), dim3(ny / NR, 1, nruns),
                           dim3(C::ATPB), 0, st, runs, sa);
      return true;
    }
    return false;
  }
  template <int NR, int E>
  static bool advf(const Run* runs, int nruns, int ny, const StepArgs* sa, bool inertial,
                   hipStream_t st) {
    return inertial ? adv<NR, 3, E>(runs, nruns, ny, sa, st)
                    : adv<NR, 2, E>(runs, nruns, ny, sa, st);
  }
  static bool flow_adv(const Run* runs, int nruns, int ny, const StepArgs* sa, bool inertial,
                       int shape, hipStream_t st) {
    switch (shape) {
      case FUSE_2N: return advf<2, EN>(runs, nruns, ny, sa, inertial, st);
      case FUSE_2W: return advf<2, EW>(runs, nruns, ny, sa, inertial, st);
      case FUSE_4W: return advf<4, EW>(runs, nruns, ny, sa, inertial, st);
    }
    return false;
  }
  template <int NR, int E>
  static bool mu(const Run* runs, int nruns, int ny, const StepArgs* sa, hipStream_t st) {
    using C = FuseCfg<T, L, NR, 2, E>;
    if constexpr (C::MOK) {
      if (nruns > 0)
        hipLaunchKernelGGL((k_phi_mu<T, 2 * L, NR, E>), dim3(ny / NR, 1, nruns), dim3(C::MTPB),
                           0, st, runs, sa);
      return true;
    }
    return false;
  }
  static bool phi_mu(const Run* runs, int nruns, int ny, const StepArgs* sa, int shape,
                     hipStream_t st) {
    switch (shape) {
      case FUSE_2N: return mu<2, EN>(runs, nruns, ny, sa, st);
      case FUSE_2W: return mu<2, EW>(runs, nruns, ny, sa, st);
      case FUSE_4W: return mu<4, EW>(runs, nruns, ny, sa, st);
    }
    return false;
  }
  static void set(Ops* o) {
    o->flow_adv = &flow_adv;
    o->phi_mu = &phi_mu;
  }
};

template <typename T>
void set_fused(int nx, Ops* o) {
  switch (nx) {
    case 8: FusedLaunch<T, 4>::set(o); break;
    case 16: FusedLaunch<T, 8>::set(o); break;
    case 32: FusedLaunch<T, 16>::set(o); break;
    case 64: FusedLaunch<T, 32>::set(o); break;
    case 128: FusedLaunch<T, 64>::set(o); break;
    case 256: FusedLaunch<T, 128>::set(o); break;
    case 512: FusedLaunch<T, 256>::set(o); break;
    case 1024: FusedLaunch<T, 512>::set(o); break;
    case 2048: FusedLaunch<T, 1024>::set(o); break;
    default: o->flow_adv = nullptr; o->phi_mu = nullptr; break;
  }
}

}  // namespace le
