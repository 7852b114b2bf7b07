// Row-pass instantiations, single precision, p = 5 and 6.
#define PF_T float
#define PF_ROW_P 5
#include "k_row.inc"
