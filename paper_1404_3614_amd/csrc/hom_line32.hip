// Register-transform passes of any length (hom_line.hpp), FP32.
#include "hom_line.hpp"

namespace hom {
namespace ln {

template bool reg_row<float>(bool, const Geo&, const UnitDev*, int, int, int, const int*, hipStream_t, hipError_t*);
template bool reg_mid<float>(const Geo&, const UnitDev*, int, int, hipStream_t, hipError_t*);
template bool reg_col<float>(const Geo&, const UnitDev*, int, int, hipStream_t, hipError_t*);

}  // namespace ln
}  // namespace hom
