// Instantiation of the 1-D / 2-D adjoint stage kernel: float, 1-D.
#include "adjoint2d.hpp"

namespace atfd {
hipError_t launch_adj1d_f32(const AdjParams& q, hipStream_t st) { return launch_adj2d<float, 1>(q, st); }
}  // namespace atfd
