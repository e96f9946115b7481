// Electron step of batches whose discharges all have three channels without
// attachment and drift-diffusion ions (k_electron.h).
#define HD_ELEC_KIND kElecDd
#include "k_electron.h"

namespace hd {
HD_ELEC_EXPORT(elec_kernel_dd)
}  // namespace hd
