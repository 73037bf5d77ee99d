// Instantiation of the 3-D adjoint stage kernel: double.
#include "adjoint3d.hpp"

namespace atfd {
hipError_t launch_adj3d_f64(const AdjParams& q, hipStream_t st) { return launch_adj3d<double>(q, st); }
}  // namespace atfd
