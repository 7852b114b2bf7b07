// One-pass strided axes of small 3D grids, single precision.
#define PF_T float
#include "k_col2.inc"
