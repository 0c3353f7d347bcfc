// Fused small-block Lanczos kernels: F64 storage, 1 vector per lane.
#include "lanczos_wg.h"

namespace ftlm {
namespace hvk {
FTLM_WG_INSTANTIATE(double, 1)
}  // namespace hvk
}  // namespace ftlm
