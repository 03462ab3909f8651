// Instances of the binned single-launch kernels for 3 tracers.
#include "tmm_bins.hpp"

namespace tmm {
TMM_BINS_KERNELS(3)
}  // namespace tmm
