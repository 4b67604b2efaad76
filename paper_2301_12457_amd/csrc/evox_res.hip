// One benchmark function's resident PSO kernels (compiled once per function
// with -DEVOX_FN=<id>).
#include "evox_pso_resident.hpp"

#ifndef EVOX_FN
#error "compile with -DEVOX_FN=<function id>"
#endif

namespace evox {

template hipError_t launch_pso_res_t<EVOX_FN>(int, const PsoResPlan &, const PsoArgs &, const PsoResArgs &, hipStream_t);

}  // namespace evox
