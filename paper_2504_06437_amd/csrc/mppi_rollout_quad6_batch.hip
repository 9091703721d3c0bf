// Batched (persistent) rollout kernels of the quad6 model, compiled in a unit of
// their own.
#include "mppi_device.hpp"

namespace dbas {

BatchRolloutKernel batch_rollout_kernel_quad6(int key) { return batch_kernel_of<MPPI_QUAD6>(key); }

}  // namespace dbas
