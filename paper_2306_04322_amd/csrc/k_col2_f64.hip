// One-pass strided axes of small 3D grids, double precision.
#define PF_T double
#include "k_col2.inc"
