// Instantiation of the plane-mapped step kernel for double-precision populations (one translation unit
// per storage type, so that the library's sources compile in parallel).
#include "step_kernel.hpp"

namespace eselbm {

hipError_t launch_step_flat_f64(int D, int mode, bool diag, const StepArgs &a, hipStream_t s)
{
    return launch_step_storage<double, true>(D, mode, diag, a, s);
}

}  // namespace eselbm
