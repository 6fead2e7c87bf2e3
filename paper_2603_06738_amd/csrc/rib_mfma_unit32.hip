// The one-kernel bf16 backward for augmented rows of up to 32 columns (see rib_mfma_unit.h).
#include "rib_mfma_unit.h"

namespace rib {
namespace unit {
hipError_t launch32(const Geo &g, const Args &a) { return unit_flags<32>(g, a); }
}  // namespace unit
}  // namespace rib
