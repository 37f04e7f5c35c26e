// The resident Jacobi-CG in FP64: kernel variants.
#include "resident_impl.hpp"

namespace pb {
namespace {
template <>
const std::vector<ResVariant>& res_variants<double>() {
    static const std::vector<ResVariant> v = {
        PB_RES_VARIANT(double, 256, 2), PB_RES_VARIANT(double, 256, 4), PB_RES_VARIANT(double, 512, 4),
        PB_RES_VARIANT(double, 512, 6), PB_RES_VARIANT(double, 512, 8), PB_RES_VARIANT(double, 512, 9),
    };
    return v;
}
}  // namespace
PB_RES_INSTANCES(double)
}  // namespace pb
