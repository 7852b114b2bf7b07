// Row-pass instantiations, double precision, p = 1 and 2 and the general kernels.
#define PF_T double
#define PF_ROW_P 1
#include "k_row.inc"
