// The resident Jacobi-CG in FP32: kernel variants.
#include "resident_impl.hpp"

namespace pb {
namespace {
template <>
const std::vector<ResVariant>& res_variants<float>() {
    static const std::vector<ResVariant> v = {
        PB_RES_VARIANT(float, 256, 2),  PB_RES_VARIANT(float, 256, 4),  PB_RES_VARIANT(float, 512, 4),
        PB_RES_VARIANT(float, 512, 6),  PB_RES_VARIANT(float, 512, 8),  PB_RES_VARIANT(float, 512, 10),
        PB_RES_VARIANT(float, 512, 12), PB_RES_VARIANT(float, 512, 14), PB_RES_VARIANT(float, 512, 19),
        PB_RES_COMPACT(24),             PB_RES_COMPACT(32),             PB_RES_COMPACT(43),
    };
    return v;
}
}  // namespace
PB_RES_INSTANCES(float)
}  // namespace pb
