// Fused small-block Lanczos kernels: F64 storage, 2 vectors per lane.
#include "lanczos_wg.h"

namespace ftlm {
namespace hvk {
FTLM_WG_INSTANTIATE(double, 2)
}  // namespace hvk
}  // namespace ftlm
