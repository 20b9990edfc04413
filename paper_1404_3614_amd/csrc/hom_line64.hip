// Register-transform passes of any length (hom_line.hpp), FP64.
#include "hom_line.hpp"

namespace hom {
namespace ln {

template bool reg_row<double>(bool, const Geo&, const UnitDev*, int, int, int, const int*, hipStream_t, hipError_t*);
template bool reg_mid<double>(const Geo&, const UnitDev*, int, int, hipStream_t, hipError_t*);
template bool reg_col<double>(const Geo&, const UnitDev*, int, int, hipStream_t, hipError_t*);
template bool reg_line<double>(Cx<double>*, int, int, int, const Cx<double>*, int, hipStream_t, hipError_t*);

// Grid values of A and A^-1 of n cells of one geometry (jobs: device table; null: the one cell
// `one`) from their Fourier data; false when an axis has no split.
bool reg_coef_setup(const int* Mz, int nc, const CoefJob* jobs, const CoefJob& one, int n,
                    const Cx<double>* const* tw, hipStream_t st, hipError_t* err) {
  if (n < 1 || n > 65535) return false;
  int ax[3], na = 0;
  for (int x = 0; x < 3; ++x)
    if (x == 2 || Mz[x] > 1) ax[na++] = x;
  LineArgs a[3];
  dim3 grid[3];
  size_t lds[3];
  for (int i = 0; i < na; ++i) {
    const int x = ax[i];
    const int outer = nc * (x > 0 ? Mz[0] : 1) * (x > 1 ? Mz[1] : 1);
    const int inner = (x < 2 ? Mz[2] : 1) * (x < 1 ? Mz[1] : 1);
    if (!array_lines<double>(outer, Mz[x], inner, &a[i], &grid[i], &lds[i])) return false;
    if (x == 2 && !a[i].rowwise) return false;
    grid[i].z = n;
  }
  for (int k = 0; k < 2; ++k)
    for (int i = 0; i < na; ++i) {
      auto go = [&]() -> hipError_t {
#define HOM_C(RM) launch_line(k_line_setup<RM>, grid[i], lds[i], st, jobs, one, a[i], tw[ax[i]], k, i == 0, i == na - 1)
        HOM_RCLASS(a[i].A, a[i].B, HOM_C);
#undef HOM_C
      };
      *err = go();
      if (*err != hipSuccess) return true;
    }
  return true;
}

}  // namespace ln
}  // namespace hom
