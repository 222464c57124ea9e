// F32 instances of the linear model's adjoint on the matrix cores.
#include "adjoint_linear.hpp"

namespace empc {
template <>
hipError_t launch_adjoint_linear<float>(const ProbView<float> &P, const float *x0, const float *knots,
                                      int64_t ncand, int64_t ld, float *dJ, float *cost, int steps,
                                      float lr, float *knots_io, float *cost_io, hipStream_t s,
                                      bool *taken) {
    return launch_adjoint_linear_t<float>(P, x0, knots, ncand, ld, dJ, cost, steps, lr, knots_io,
                                        cost_io, s, taken);
}
}  // namespace empc
