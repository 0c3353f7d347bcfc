// Fused small-block Lanczos kernels: F64 storage, 4 vectors per lane.
#include "lanczos_wg.h"

namespace ftlm {
namespace hvk {
FTLM_WG_INSTANTIATE(double, 4)
}  // namespace hvk
}  // namespace ftlm
