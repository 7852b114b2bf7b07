// Row-pass instantiations, double precision, p = 5 and 6.
#define PF_T double
#define PF_ROW_P 5
#include "k_row.inc"
