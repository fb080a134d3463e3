// Multi-factor passes in registers over the systems of many operators, complex128.
#include "zrows_multi.h"

namespace hfci {
template bool MultiLaunch<double2>::factor_rows(hipStream_t, const RowsClass&, const MultiInst*, const RowsShape*,
                                               const MultiSys<double2>*, const int2*, int, int, int, int, int, int, int,
                                               int);
template bool MultiLaunch<double2>::rows_class(const std::vector<GridDesc>&, const std::vector<double>&,
                                              const std::vector<double>&, RowsClass*, std::vector<RowsShape>*);
}  // namespace hfci
