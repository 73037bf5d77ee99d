// Instantiation of the 3-D adjoint stage kernel: float.
#include "adjoint3d.hpp"

namespace atfd {
hipError_t launch_adj3d_f32(const AdjParams& q, hipStream_t st) { return launch_adj3d<float>(q, st); }
}  // namespace atfd
