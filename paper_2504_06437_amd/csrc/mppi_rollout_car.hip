// Standalone rollout kernels of the car model, compiled in a unit of their own.
#include "mppi_device.hpp"

namespace dbas {

hipError_t launch_rollout_car(const DevParams& p, const StepArgs& a, size_t lds, hipStream_t s)
{
    return launch_rollout_m<MPPI_CAR>(p, a, lds, s);
}

}  // namespace dbas
