// Layout of the x-spectra (pf_kernels.h describes both): strides, and the rules
// that choose between them for a grid.  Host code.
#pragma once

#include <cstddef>

#include "pf_kernels.h"

namespace pf {

struct SpecLayout {
  int rs, ts;     // row and tile stride
  long long nyo;  // offset of the Nyquist values within a field
  size_t field;   // complex elements per field
};

// Complex elements of the Nyquist array of a field (128-byte multiple).
inline size_t nyquist_elements(int rows, bool f32) {
  const size_t al = f32 ? 16 : 8;  // complex values per 128 bytes
  return (size_t(rows) + al - 1) / al * al;
}

// x-spectrum rows hold kx = 0 .. Nx/2 - 1; the Nyquist values follow the
// rows as one array per field, in both layouts.  Row-major 2D rows carry
// one more 128-byte segment: the column pass strides along y by the row
// length, and a power-of-two row stride made its concurrent accesses
// collide (1024^2 FP32 column pass 17.7 -> 16.5 us), except float rows of
// 4096 points, where the unpadded 16 KiB stride measured faster.  3D rows
// (and planes) are not padded: no gain was measured there.
inline SpecLayout row_major_spectra(int ndim, int nx, int rows, bool f32) {
  const int al = f32 ? 16 : 8;
  SpecLayout l;
  l.rs = (nx / 2 + al - 1) / al * al;
  if (ndim == 2 && !(f32 && nx == 4096)) l.rs += al;
  l.ts = f32 ? KTile<float>::N : KTile<double>::N;
  l.nyo = (long long)rows * l.rs;
  l.field = size_t(l.nyo) + nyquist_elements(rows, f32);
  return l;
}

inline SpecLayout tiled_spectra(int nx, int rows, bool f32) {
  SpecLayout l;
  l.rs = f32 ? KTile<float>::N : KTile<double>::N;
  l.ts = l.rs * rows;
  l.nyo = (long long)(nx / 2) * rows;
  l.field = size_t(l.nyo) + nyquist_elements(rows, f32);
  return l;
}

// 3D grids whose strided axes go in one pass (k_col2.inc): few points per (y, z)
// plane, so that a work-group holds the planes of a few columns; above 1024
// points a work-group holds one column, which pays only while there are few of
// them.  FS step, four launches / two, us:
//   up to 1024 points, F = 5: FP32 16^3 13.3 / 8.3, 32^3 15.0 / 10.5, 1024 x 32 x 32
//   41.8 / 37.5; FP64 32^3 16.2 / 11.7, 1024 x 32 x 32 74.9 / 54.2
//   up to 2048, FP32 (64 x 32 planes): nx = 8 a third less for every F; nx = 128,
//   F = 2 .. 9, 1.07 to 1.25 times as fast (one-step call 1.00 to 1.12); nx = 256
//   1.07 (F = 2) to 0.87 (F = 9); nx = 512 0.90 to 0.79.
//   FP64: nx = 512 1.09 (F = 2) to 1.00 (F = 9); nx = 1024 1.05, 1.05, 1.03 (F = 2 .. 4),
//   1.01 with the one-step call 0.93 (F = 5 .. 7), 0.90 (F = 8), 0.94 (F = 9)
//   up to 4096 (64 x 64 planes): FP32 64^3 1.02 to 1.15 (F = 2 .. 8), 0.98 (F = 9); 128 x
//   64 x 64 0.92 to 1.11.  FP64 64^3 1.03 to 1.20 (F = 2 .. 7), 0.97 (F = 9); nx <= 32
//   with F < 4 0.94 to 1.00 (one-step call 0.86 to 0.95), with F >= 4 1.00 to 1.22
inline bool one_pass_strided(int nx, int rows, int F, bool f32) {
  if (rows <= 1024) return true;
  if (rows <= 2048) return f32 ? nx <= 128 : nx * F <= 4608;
  return rows <= PF_COL2_MAX && nx * F <= 320 && (f32 || nx > 32 || F >= 4);
}

// 2D grids with the tiled x-spectrum layout (pf_kernels.h).  A compute unit
// fetches whole 128-byte lines, of which a column work-group of two or four
// columns used 16 or 32 bytes in the row-major layout; the row passes pay for
// the tiles where their work-groups are few.  FS step, F = 5, row-major / tiled:
//   FP32 4096^2 649 / 549 us, 2048^2 125 / 103, 1024 x 2048 60.8 / 51.1, 512 x
//   2048 38.2 / 33.8, 512 x 1024 27.7 / 26.4, 64 x 1024 14.4 / 12.1; but 1024^2
//   31.6 / 33.1, 512^2 16.9 / 18.5
//   FP64 4096^2 1420 / 1198, 2048^2 262 / 244, 1024^2 53.7 / 52.9, 2048 x 512
//   59.1 / 55.0; but 1024 x 512 31.2 / 32.8, and 512^2 25.1 / 24 or 31 by the
//   place of the buffers in memory
// With more than four order parameters the line of 1024-point rows lies higher:
// p = 8, FP64 1024^2 99 / 104, FP32 1024 x 2048 95 / 94 with the one-step call 0.95 and
// the energy 0.91 times as fast (p = 5 and 6, on which tiles measured 1.16 times
// as fast, go with p = 8).  One or more lines of padding per tile: no
// faster (2048^2 FP64 244 / 252, 4096^2 FP32 549 / 552, 1024^2 FP64 52.9 / 54).
inline bool tiled_layout(int ndim, int nx, int ny, int p, bool f32) {
  if (ndim != 2) return false;
  const bool few = p <= 4;
  if (ny >= 2048) return few || !f32 || nx != 1024;
  if (f32) return ny >= 1024 && nx <= 512;
  if (ny >= 1024) return few || nx != 1024;
  return ny >= 512 && few && nx >= 2048;
}

// FP64 grids with the tiled layout whose adjoint steps and whose spectral energy
// are done row-major all the same (neither carries a spectrum from the FS steps):
// their row passes are one row per work-group, pieces of 32 bytes in a tile, and
// their column passes gain less.  Adjoint step, row-major / tiled, us: 4096 x 1024
// p = 2 421 / 457, p = 6 1296 / 1377, 4096 x 2048 p = 2 836 / 892, 2048 x 1024 p = 6 498 /
// 535, p = 8 742 / 813; but 4096 x 512 p = 2 218 / 212, 2048 x 1024 p = 4 285 / 281, 2048^2
// p = 6 1022 / 1024.  Energy: 1024 x 4096 p = 4 238 / 271, p = 5 291 / 319, 1024 x 2048
// p = 8 237 / 250; but 1024 x 4096 p = 3 164 / 156, 1024 x 2048 p = 7 186 / 182, 2048 x
// 4096 p = 2 247 / 210.
inline bool adjoint_row_major(int nx, int ny, int p, bool f32) {
  return !f32 && ((nx == 4096 && ny >= 1024) || (nx == 2048 && ny == 1024 && p >= 6));
}
inline bool energy_row_major(int nx, int ny, int F, bool f32) { return !f32 && nx == 1024 && ny * F >= 18432; }

}  // namespace pf
