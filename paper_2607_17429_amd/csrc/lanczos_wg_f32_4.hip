// Fused small-block Lanczos kernels: F32 storage, 4 vectors per lane.
#include "lanczos_wg.h"

namespace ftlm {
namespace hvk {
FTLM_WG_INSTANTIATE(float, 4)
}  // namespace hvk
}  // namespace ftlm
