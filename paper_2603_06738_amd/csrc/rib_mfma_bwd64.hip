// The bf16 backward kernels for augmented rows of up to 64 columns (see rib_mfma_bwd.h).
#include "rib_mfma_bwd.h"

namespace rib {
namespace bwd {
hipError_t launch64(const Geo &g, const Args &a) { return launch_flags<64>(g, a); }
}  // namespace bwd
}  // namespace rib
