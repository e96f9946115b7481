// Electron step of any batch, and the choice and launch of the electron
// kernels (k_electron.h).
#define HD_ELEC_KIND kElecAny
#include "k_electron.h"

#include <algorithm>

namespace hd {

HD_ELEC_EXPORT(elec_kernel_any)
const void* elec_kernel_dd(bool f64, int variant);
const void* elec_kernel_full(bool f64, int variant);

static const void* elec_kernel_of(int kind, bool f64, int variant) {
  return kind == kElecDd ? elec_kernel_dd(f64, variant)
         : kind == kElecFull ? elec_kernel_full(f64, variant)
                             : elec_kernel_any(f64, variant);
}

// Variant v < kElecWide: kernel v with kElecThreads per workgroup;
// kElecWide + v: its wide twin with kElecThreadsWide.  The FP64 kernels and the
// register-prefetch kernel have none and those variants are rejected: in FP64
// sixteen waves' collision queues take 96 KB, which leaves no room for the
// arrays of the large grids that wide workgroups are for, and the prefetch
// kernel is for few waves.  Registers would allow most of them (97 to 102 VGPRs
// of 128; 141 to 144 for FP64 with the prefetch).
inline int elec_threads(int variant) {
  return variant >= kElecWide ? kElecThreadsWide : kElecThreads;
}

template <class P>
size_t electron_lds_bytes(int D, int tab_max, int nn_max, int nb1_max, int fluid_nn, int K_max,
                          int variant) {
  return lds_layout<P>(elec_args<P>(D, tab_max, nn_max, nb1_max, fluid_nn, K_max,
                                    elec_threads(variant) / 64)).total;
}

template <class P>
hipError_t launch_electron_impl(const Disch<P>* d_dev, int D, int grid, int tab_max, int nn_max,
                                int nb1_max, int fluid_nn, int K_max, int variant, int kind, hipStream_t s) {
  if (variant < 0 || variant >= kElecVariants) return hipErrorInvalidValue;
  const int nt = elec_threads(variant);
  const ElecArgs a = elec_args<P>(D, tab_max, nn_max, nb1_max, fluid_nn, K_max, nt / 64);
  const size_t lds = lds_layout<P>(a).total;
  const void* fk = elec_kernel_of(kind, sizeof(P) == 8, variant);
  if (!fk) return hipErrorInvalidValue;
  const Disch<P>* ds = d_dev;
  ElecArgs args = a;
  void* av[2] = {&ds, &args};
  args.groups = grid;
  grid = (int)launch_groups((uint32_t)D, (uint32_t)grid);
  return hipLaunchKernel(fk, dim3(grid), dim3(nt), av, lds, s);
}

template <class P>
int electron_occupancy(int tab_max, int nn_max, int nb1_max, int fluid_nn, int K_max, int D,
                       int variant, int kind) {
  int nb = 0;
  if (variant < 0 || variant >= kElecVariants) return 0;
  const size_t lds = electron_lds_bytes<P>(D, tab_max, nn_max, nb1_max, fluid_nn, K_max, variant);
  const void* fk = elec_kernel_of(kind, sizeof(P) == 8, variant);
  if (!fk) return 0;  // no wide twin
  if (hipFuncSetAttribute(fk, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) !=
          hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fk, elec_threads(variant), lds) !=
          hipSuccess) {
    (void)hipGetLastError();  // an answer, not an error for the next launch to report
    return 0;
  }
  // Sixteen waves per CU: on small grids, where the LDS has room for a third
  // narrow workgroup, work divided for three per CU is slower (64 discharges
  // of 16,384 electrons 39.8 us per step instead of 35.0).
  return std::min(nb, 16 * 64 / elec_threads(variant));
}

int electron_variants() { return kElecVariants; }

template size_t electron_lds_bytes<float>(int, int, int, int, int, int, int);
template size_t electron_lds_bytes<double>(int, int, int, int, int, int, int);
template hipError_t launch_electron_impl<float>(const Disch<float>*, int, int, int, int, int, int,
                                                int, int, int, hipStream_t);
template hipError_t launch_electron_impl<double>(const Disch<double>*, int, int, int, int, int,
                                                 int, int, int, int, hipStream_t);
template int electron_occupancy<float>(int, int, int, int, int, int, int, int);
template int electron_occupancy<double>(int, int, int, int, int, int, int, int);

}  // namespace hd
