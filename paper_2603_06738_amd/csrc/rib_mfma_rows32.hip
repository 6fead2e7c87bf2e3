// The bf16 forward kernels for windows of any size, augmented rows of up to 32 columns (see rib_mfma_rows.h).
#include "rib_mfma_rows.h"

namespace rib {
namespace fwd_rows {
hipError_t launch32(const Geo &g, int qb, const Args &a) { return launch_flags<32>(g, qb, a); }
}  // namespace fwd_rows
}  // namespace rib
