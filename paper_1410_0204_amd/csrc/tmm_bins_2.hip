// Instances of the binned single-launch kernels for 2 tracers.
#include "tmm_bins.hpp"

namespace tmm {
TMM_BINS_KERNELS(2)
}  // namespace tmm
