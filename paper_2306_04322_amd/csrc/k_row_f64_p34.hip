// Row-pass instantiations, double precision, p = 3 and 4.
#define PF_T double
#define PF_ROW_P 3
#include "k_row.inc"
