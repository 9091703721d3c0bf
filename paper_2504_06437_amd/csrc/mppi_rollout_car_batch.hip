// Batched (persistent) rollout kernels of the car model, compiled in a unit of
// their own.
#include "mppi_device.hpp"

namespace dbas {

BatchRolloutKernel batch_rollout_kernel_car(int key) { return batch_kernel_of<MPPI_CAR>(key); }

}  // namespace dbas
