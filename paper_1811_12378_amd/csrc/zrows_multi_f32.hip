// Multi-factor passes in registers over the systems of many operators, complex64.
#include "zrows_multi.h"

namespace hfci {
template bool MultiLaunch<float2>::factor_rows(hipStream_t, const RowsClass&, const MultiInst*, const RowsShape*,
                                               const MultiSys<float2>*, const int2*, int, int, int, int, int, int, int,
                                               int);
template bool MultiLaunch<float2>::rows_class(const std::vector<GridDesc>&, const std::vector<double>&,
                                              const std::vector<double>&, RowsClass*, std::vector<RowsShape>*);
}  // namespace hfci
