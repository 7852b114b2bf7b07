// Row-pass instantiations, single precision, p = 1 and 2 and the general kernels.
#define PF_T float
#define PF_ROW_P 1
#include "k_row.inc"
