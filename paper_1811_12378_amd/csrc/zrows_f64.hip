// Multi-factor passes with planes in registers (zrows.h), complex128.
#include "zrows_launch.h"

namespace hfci {
template bool Launch<double2>::factor_rows(hipStream_t, const GridDesc&, const void*, const FactorArgs<double2>&, int, int,
                                          const RowsShape&);
template RowsShape Launch<double2>::rows_shape(const GridDesc&, int, int, int);
template bool Launch<double2>::rows_fits(const GridDesc&);
template bool Launch<double2>::rows_run(const GridDesc&);
}  // namespace hfci
