// Electron step of batches whose discharges all have three channels without
// attachment and the full ion fluid (k_electron.h).
#define HD_ELEC_KIND kElecFull
#include "k_electron.h"

namespace hd {
HD_ELEC_EXPORT(elec_kernel_full)
}  // namespace hd
