// Row-pass instantiations, single precision, p = 7 and 8.
#define PF_T float
#define PF_ROW_P 7
#include "k_row.inc"
