// Instances of the binned single-launch kernels for 1 tracer.
#include "tmm_bins.hpp"

namespace tmm {
TMM_BINS_KERNELS(1)
}  // namespace tmm
