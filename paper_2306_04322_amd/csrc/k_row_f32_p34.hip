// Row-pass instantiations, single precision, p = 3 and 4.
#define PF_T float
#define PF_ROW_P 3
#include "k_row.inc"
