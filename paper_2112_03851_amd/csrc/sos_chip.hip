// Launches of the on-chip fused CG kernel (sos_chip.h) for one set of
// variants, SOS_CHIP_SET (compiled once per value), and their dispatch
// (SOS_CHIP_SET 0); all sets in one unit with SOS_CHIP_SET -1.
#include "sos_chip.h"

#ifndef SOS_CHIP_SET
#error SOS_CHIP_SET must be defined (0..5, or -1)
#endif

namespace sos {

template <typename T, int P, bool Q, bool WL>
static hipError_t chip_one(const Dev& d, const SegLaunch& L, int threads, const FusedArgs& a, hipStream_t st,
                           int* per_cu) {
  if (per_cu)
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, (const void*)k_chip_cg<T, P, Q, WL>, threads,
                                                        a.lds_bytes);
  hipLaunchKernelGGL((k_chip_cg<T, P, Q, WL>), dim3(a.n_teams * a.team), dim3(threads), a.lds_bytes, st, d,
                     L.bfirst, a);
  return hipGetLastError();
}

template <typename T, int P, bool WL>
static hipError_t chip_q(const Dev& d, const SegLaunch& L, int threads, const FusedArgs& a, hipStream_t st,
                          int* per_cu) {
  if (a.chip_planes != P || (a.chip_wl != 0) != WL) return hipErrorInvalidValue;
  return d.hasq ? chip_one<T, P, true, WL>(d, L, threads, a, st, per_cu)
                : chip_one<T, P, false, WL>(d, L, threads, a, st, per_cu);
}

// One set of variants (each set compiled in a translation unit of its own).
template <int SET>
hipError_t launch_chip_set(const Dev& d, const SegLaunch& L, int threads, const FusedArgs& a, hipStream_t st,
                           int* per_cu) {
  if constexpr (SET == 0) return chip_q<float, 17, false>(d, L, threads, a, st, per_cu);
  else if constexpr (SET == 1) return chip_q<float, 17, true>(d, L, threads, a, st, per_cu);
  else if constexpr (SET == 2) return chip_q<float, 9, true>(d, L, threads, a, st, per_cu);
  else if constexpr (SET == 3) return chip_q<float, 5, true>(d, L, threads, a, st, per_cu);
  else if constexpr (SET == 4) return chip_q<double, 5, true>(d, L, threads, a, st, per_cu);
  else return chip_q<float, 12, true>(d, L, threads, a, st, per_cu);
}

#define SOS_CHIP_DECL(PREFIX, SET)                                                                      \
  PREFIX template hipError_t launch_chip_set<SET>(const Dev&, const SegLaunch&, int, const FusedArgs&, \
                                                  hipStream_t, int*);

#if SOS_CHIP_SET > 0
SOS_CHIP_DECL(, SOS_CHIP_SET)
#endif

// The first unit also dispatches (the only one with SOS_CHIP_SET -1: all sets).
#if SOS_CHIP_SET <= 0
#if SOS_CHIP_SET == 0
SOS_CHIP_DECL(extern, 1)
SOS_CHIP_DECL(extern, 2)
SOS_CHIP_DECL(extern, 3)
SOS_CHIP_DECL(extern, 4)
SOS_CHIP_DECL(extern, 5)
#endif

hipError_t launch_chip(const Dev& d, const SegLaunch& L, int fp32, int threads, const FusedArgs& a, hipStream_t st,
                       int* per_cu) {
  if (threads > kChipThreads || a.team < 1 || a.n_teams < (per_cu ? 0 : 1)) return hipErrorInvalidValue;
  if (!fp32) return launch_chip_set<4>(d, L, threads, a, st, per_cu);
  if (a.chip_planes == 17)
    return a.chip_wl ? launch_chip_set<1>(d, L, threads, a, st, per_cu)
                     : launch_chip_set<0>(d, L, threads, a, st, per_cu);
  if (a.chip_planes == 12) return launch_chip_set<5>(d, L, threads, a, st, per_cu);
  return a.chip_planes == 9 ? launch_chip_set<2>(d, L, threads, a, st, per_cu)
                            : launch_chip_set<3>(d, L, threads, a, st, per_cu);
}
#endif

}  // namespace sos
