// F64 instances of the linear model's adjoint on the matrix cores.
#include "adjoint_linear.hpp"

namespace empc {
template <>
hipError_t launch_adjoint_linear<double>(const ProbView<double> &P, const double *x0, const double *knots,
                                      int64_t ncand, int64_t ld, double *dJ, double *cost, int steps,
                                      double lr, double *knots_io, double *cost_io, hipStream_t s,
                                      bool *taken) {
    return launch_adjoint_linear_t<double>(P, x0, knots, ncand, ld, dJ, cost, steps, lr, knots_io,
                                        cost_io, s, taken);
}
}  // namespace empc
