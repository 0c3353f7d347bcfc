// Fused small-block Lanczos kernels: F32 storage, 3 vectors per lane.
#include "lanczos_wg.h"

namespace ftlm {
namespace hvk {
FTLM_WG_INSTANTIATE(float, 3)
}  // namespace hvk
}  // namespace ftlm
