// Batched (persistent) rollout kernels of the quad5 model, compiled in a unit of
// their own.
#include "mppi_device.hpp"

namespace dbas {

BatchRolloutKernel batch_rollout_kernel_quad5(int key) { return batch_kernel_of<MPPI_QUAD5>(key); }

}  // namespace dbas
