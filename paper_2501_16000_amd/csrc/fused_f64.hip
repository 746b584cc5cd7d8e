// fused_f64.hip -- the fused multi-step sweeps of lb_step for
// FP64 storage: instantiations of fused_impl.hpp.
#include "fused_impl.hpp"

namespace oreg {

template hipError_t fused_launch_st<LB_F64>(int, int, int, const void*, void*, const Geometry&,
                                           const Coef64&, int, int, int, const unsigned int*,
                                           unsigned int*, hipStream_t);
template hipError_t fused_occupancy_st<LB_F64>(int, int, int*);

}  // namespace oreg
