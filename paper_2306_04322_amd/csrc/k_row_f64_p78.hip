// Row-pass instantiations, double precision, p = 7 and 8.
#define PF_T double
#define PF_ROW_P 7
#include "k_row.inc"
