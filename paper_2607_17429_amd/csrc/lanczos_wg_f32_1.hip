// Fused small-block Lanczos kernels: F32 storage, 1 vector per lane.
#include "lanczos_wg.h"

namespace ftlm {
namespace hvk {
FTLM_WG_INSTANTIATE(float, 1)
}  // namespace hvk
}  // namespace ftlm
