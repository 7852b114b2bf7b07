// Explicit finite-difference comparison step (forward Euler, 5-point /
// 7-point periodic Laplacian, every right-hand side at time t) and the
// forward-difference free-energy sums.
//
// Most grids take a fused step (fd2_fused_kernel, fd3_march_kernel,
// fd3_tile_kernel): one launch per step, mu = df/dc - kappa_c lap(c) kept on
// the chip.  The other 3D grids (fd_fused has the rule) take two kernels with
// mu in memory between them.
//
// Every kernel gives a thread V consecutive points along x, read as one vector
// of up to 16 bytes (V = 4 float or 2 double on large grids, fewer on small
// ones): each field's centre values and its y / z neighbours arrive as one
// vector load each, the x neighbours inside the vector come from registers
// and only the two at its ends are extra scalar loads, so a field costs 5
// (2D) or 7 (3D) loads per V points instead of per point.  The y and z
// neighbours are rows that neighbouring work-groups also read; each XCD takes
// a contiguous band of the grid so those re-reads stay in its own L2.  On
// larger 3D grids each thread instead marches along z over a few planes and
// keeps its neighbour planes in registers, and a work-group stages the
// current plane of its rows (plus halo rows) in LDS for the y and x
// neighbours.  Periodic wrap uses power-of-two masks instead of ghost layers.
#include "pf_kernels.h"
#include "pf_launch.h"

namespace pf {

// V consecutive points of one row, loaded and stored as one aligned vector
// (V * sizeof(T) <= 16 bytes).
template <typename T, int V>
struct alignas(sizeof(T) * V) FdVec {
  T v[V];
};

template <typename T, int V>
__device__ __forceinline__ FdVec<T, V> ld_vec(const T* __restrict__ p) {
  return *reinterpret_cast<const FdVec<T, V>*>(p);
}

template <typename T, int V>
__device__ __forceinline__ void st_vec(T* p, const T* v) {
  FdVec<T, V> w;
#pragma unroll
  for (int k = 0; k < V; ++k) w.v[k] = v[k];
  *reinterpret_cast<FdVec<T, V>*>(p) = w;
}

// The same store with the non-temporal hint: the marching kernels write
// their outputs once and never read them back, so the stores should not
// displace the neighbour planes the kernel re-reads from L2.
template <typename T, int V>
__device__ __forceinline__ void st_vec_nt(T* p, const T* v) {
  if constexpr (V == 1) {
    __builtin_nontemporal_store(v[0], p);
  } else {
    typedef T vt __attribute__((ext_vector_type(V)));
    vt w;
#pragma unroll
    for (int k = 0; k < V; ++k) w[k] = v[k];
    __builtin_nontemporal_store(w, reinterpret_cast<vt*>(p));
  }
}

// Neighbour offsets of the vector starting at point i0 (x0 = i0 mod nx, a
// multiple of V): the y and z neighbour vectors and the two x neighbours
// just outside the vector.
struct NbV {
  long long ym, yp, zm, zp, xl, xr;
};

template <typename T, int V>
__device__ __forceinline__ NbV neighbours_vec(const FdArgs<T>& a, long long i0) {
  const int x0 = int(i0 & (a.nx - 1));
  const int y = int((i0 >> a.lx) & (a.ny - 1));
  const int z = int(i0 >> (a.lx + a.ly));
  const long long row = i0 - x0;
  const long long plane = (long long)a.nx * a.ny;
  const long long zoff = (long long)z * plane;
  NbV n;
  n.xl = row + ((x0 - 1) & (a.nx - 1));
  n.xr = row + ((x0 + V) & (a.nx - 1));
  n.ym = zoff + (long long)((y - 1) & (a.ny - 1)) * a.nx + x0;
  n.yp = zoff + (long long)((y + 1) & (a.ny - 1)) * a.nx + x0;
  if (a.ndim == 3) {
    const long long rest = (long long)y * a.nx + x0;
    n.zm = (long long)((z - 1) & (a.nz - 1)) * plane + rest;
    n.zp = (long long)((z + 1) & (a.nz - 1)) * plane + rest;
  } else {
    n.zm = n.zp = i0;
  }
  return n;
}

// Laplacian of field v at the V points of the vector (centre values cv) in
// 2D, and in 3D.
template <typename T, int V>
__device__ __forceinline__ void lap_vec2(const T* __restrict__ v, const FdVec<T, V>& cv, const NbV& n,
                                         const FdArgs<T>& a, T* out) {
  const FdVec<T, V> ym = ld_vec<T, V>(v + n.ym), yp = ld_vec<T, V>(v + n.yp);
  const T xl = v[n.xl], xr = v[n.xr];
#pragma unroll
  for (int k = 0; k < V; ++k) {
    const T c = cv.v[k];
    const T left = k == 0 ? xl : cv.v[k - 1];
    const T right = k == V - 1 ? xr : cv.v[k + 1];
    out[k] = (right - T(2) * c + left) * a.ix2 + (yp.v[k] - T(2) * c + ym.v[k]) * a.iy2;
  }
}

template <typename T, int V>
__device__ __forceinline__ void lap_vec3(const T* __restrict__ v, const FdVec<T, V>& cv, const NbV& n,
                                         const FdArgs<T>& a, T* out) {
  const FdVec<T, V> ym = ld_vec<T, V>(v + n.ym), yp = ld_vec<T, V>(v + n.yp);
  const T xl = v[n.xl], xr = v[n.xr];
  // (always true here: the branch keeps the compiler from moving the loads of
  // all fields to the top, 256 x 128^2, F = 5, FP32 two-kernel step 49.0 ->
  // 44.4 us)
  FdVec<T, V> zm, zp;
  if (a.ndim == 3) {
    zm = ld_vec<T, V>(v + n.zm);
    zp = ld_vec<T, V>(v + n.zp);
  }
#pragma unroll
  for (int k = 0; k < V; ++k) {
    const T c = cv.v[k];
    const T left = k == 0 ? xl : cv.v[k - 1];
    const T right = k == V - 1 ? xr : cv.v[k + 1];
    T r = (right - T(2) * c + left) * a.ix2 + (yp.v[k] - T(2) * c + ym.v[k]) * a.iy2;
    if (a.ndim == 3) r += (zp.v[k] - T(2) * c + zm.v[k]) * a.iz2;
    out[k] = r;
  }
}

// First point of this thread's vector.  Work-groups are dealt to the eight
// XCDs round-robin; XCD x takes the x-th contiguous eighth of the grid (the
// launch rounds the group count up to a multiple of 8), so the neighbour rows
// or planes a group reads were mostly brought into that XCD's L2 by its
// neighbouring groups.
template <int V>
__device__ __forceinline__ long long fd_first_point() {
  const unsigned b = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  return ((long long)b * blockDim.x + threadIdx.x) * V;
}

// mu = df/dc - kappa_c lap(c);  eta_i' = eta_i - dt L (df/deta_i - kappa_eta lap(eta_i))
// FIXF: all PMAX order parameters in use (p fixed at compile time), as in
// the mu kernels below.
template <typename T, int PMAX, int V, bool FIXF = false>
__global__ void __launch_bounds__(256) fd_mu_kernel(FdArgs<T> a) {
  const long long i0 = fd_first_point<V>();
  if (i0 >= a.P) return;
  const NbV n = neighbours_vec<T, V>(a, i0);
  const int p = FIXF ? PMAX : a.F - 1;
  const FdVec<T, V> cc = ld_vec<T, V>(a.in + i0);
  FdVec<T, V> ce[PMAX];
#pragma unroll
  for (int j = 0; j < PMAX; ++j)
    if (j < p) ce[j] = ld_vec<T, V>(a.in + (j + 1) * a.P + i0);
  T gc[V], ge[PMAX][V];
#pragma unroll
  for (int k = 0; k < V; ++k) {
    T eta[PMAX], g[PMAX];
#pragma unroll
    for (int j = 0; j < PMAX; ++j) {
      eta[j] = (j < p) ? ce[j].v[k] : T(0);
      g[j] = T(0);
    }
    fe_grad<T, PMAX>(a.fe, p, cc.v[k], eta, gc[k], g);
#pragma unroll
    for (int j = 0; j < PMAX; ++j) ge[j][k] = g[j];
  }
  T l[V], o[V];
  lap_vec3<T, V>(a.in, cc, n, a, l);
#pragma unroll
  for (int k = 0; k < V; ++k) o[k] = gc[k] - a.kc * l[k];
  st_vec<T, V>(a.mu + i0, o);
#pragma unroll
  for (int j = 0; j < PMAX; ++j)
    if (j < p) {
      const T* e = a.in + (j + 1) * a.P;
      lap_vec3<T, V>(e, ce[j], n, a, l);
#pragma unroll
      for (int k = 0; k < V; ++k) o[k] = ce[j].v[k] - a.dtL * (ge[j][k] - a.ke * l[k]);
      st_vec<T, V>(a.out + (j + 1) * a.P + i0, o);
    }
}

// c' = c + dt M lap(mu)
template <typename T, int V>
__global__ void __launch_bounds__(256) fd_c_kernel(FdArgs<T> a) {
  const long long i0 = fd_first_point<V>();
  if (i0 >= a.P) return;
  const NbV n = neighbours_vec<T, V>(a, i0);
  const FdVec<T, V> cm = ld_vec<T, V>(a.mu + i0);
  const FdVec<T, V> c = ld_vec<T, V>(a.in + i0);
  T l[V], o[V];
  lap_vec3<T, V>(a.mu, cm, n, a, l);
#pragma unroll
  for (int k = 0; k < V; ++k) o[k] = c.v[k] + a.dtM * l[k];
  st_vec<T, V>(a.out + i0, o);
}

// 3D grids whose neighbour planes do not fit in L2: each thread takes V
// consecutive x points of one (y, x) column and marches over ZB consecutive
// planes, keeping the planes z - 1, z and z + 1 of every field it reads in
// registers, so a thread loads each of its planes once per block of ZB
// planes instead of three times.  Same arithmetic, in the same order, as
// the one-plane kernels.
template <typename T, int V>
__device__ __forceinline__ void lap_vec_z(const T* __restrict__ v, const FdVec<T, V>& zm,
                                          const FdVec<T, V>& cv, const FdVec<T, V>& zp,
                                          long long row, int x0, long long ym, long long yp,
                                          const FdArgs<T>& a, T* out) {
  const FdVec<T, V> vm = ld_vec<T, V>(v + ym), vp = ld_vec<T, V>(v + yp);
  const T xl = v[row + ((x0 - 1) & (a.nx - 1))], xr = v[row + ((x0 + V) & (a.nx - 1))];
#pragma unroll
  for (int k = 0; k < V; ++k) {
    const T c = cv.v[k];
    const T left = k == 0 ? xl : cv.v[k - 1];
    const T right = k == V - 1 ? xr : cv.v[k + 1];
    T r = (right - T(2) * c + left) * a.ix2 + (vp.v[k] - T(2) * c + vm.v[k]) * a.iy2;
    r += (zp.v[k] - T(2) * c + zm.v[k]) * a.iz2;
    out[k] = r;
  }
}

struct ZCol {
  long long plane, rest, ymr, ypr;  // plane size; (y, x0) offset in a plane; y -/+ 1 rows
  int x0, z0;
};

// Work-groups are dealt to the eight XCDs round-robin; block b is mapped to
// the logical block of XCD b % 8's contiguous eighth of the grid (the launch
// rounds the group count up to a multiple of 8), so the groups of one z
// block that hold y-adjacent rows run on one XCD and find each other's rows
// (their y neighbours) in that XCD's L2.
template <typename T, int V>
__device__ __forceinline__ bool zcol(const FdArgs<T>& a, int zb, ZCol& q) {
  const long long nxv = a.nx / V;
  const long long per = nxv * a.ny;  // vectors per plane
  const unsigned b = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  const long long t = (long long)b * blockDim.x + threadIdx.x;
  if (t >= per * (a.nz / zb)) return false;
  const long long vin = t % per;
  q.z0 = int(t / per) * zb;
  q.x0 = int(vin % nxv) * V;
  const int y = int(vin / nxv);
  q.plane = (long long)a.nx * a.ny;
  q.rest = (long long)y * a.nx + q.x0;
  q.ymr = (long long)((y - 1) & (a.ny - 1)) * a.nx + q.x0;
  q.ypr = (long long)((y + 1) & (a.ny - 1)) * a.nx + q.x0;
  return true;
}

template <typename T, int PMAX, int V, bool FIXF = false>
__global__ void __launch_bounds__(256) fd_mu_z_kernel(FdArgs<T> a, int zb) {
  ZCol q;
  if (!zcol<T, V>(a, zb, q)) return;
  const int p = FIXF ? PMAX : a.F - 1;
  FdVec<T, V> m[PMAX + 1], c[PMAX + 1], n[PMAX + 1];
  const long long zm0 = (long long)((q.z0 - 1) & (a.nz - 1)) * q.plane + q.rest;
  const long long zc0 = (long long)q.z0 * q.plane + q.rest;
#pragma unroll
  for (int f = 0; f <= PMAX; ++f)
    if (f <= p) {
      m[f] = ld_vec<T, V>(a.in + f * a.P + zm0);
      c[f] = ld_vec<T, V>(a.in + f * a.P + zc0);
    }
  for (int k = 0; k < zb; ++k) {
    const int z = q.z0 + k;
    const long long zoff = (long long)z * q.plane;
    const long long i0 = zoff + q.rest;
    const long long zn = (long long)((z + 1) & (a.nz - 1)) * q.plane + q.rest;
#pragma unroll
    for (int f = 0; f <= PMAX; ++f)
      if (f <= p) n[f] = ld_vec<T, V>(a.in + f * a.P + zn);
    T gc[V], ge[PMAX][V];
#pragma unroll
    for (int e = 0; e < V; ++e) {
      T eta[PMAX], g[PMAX];
#pragma unroll
      for (int j = 0; j < PMAX; ++j) {
        eta[j] = (j < p) ? c[j + 1].v[e] : T(0);
        g[j] = T(0);
      }
      fe_grad<T, PMAX>(a.fe, p, c[0].v[e], eta, gc[e], g);
#pragma unroll
      for (int j = 0; j < PMAX; ++j) ge[j][e] = g[j];
    }
    const long long row = zoff + (q.rest - q.x0);
    T l[V], o[V];
    lap_vec_z<T, V>(a.in, m[0], c[0], n[0], row, q.x0, zoff + q.ymr, zoff + q.ypr, a, l);
#pragma unroll
    for (int e = 0; e < V; ++e) o[e] = gc[e] - a.kc * l[e];
    st_vec_nt<T, V>(a.mu + i0, o);
#pragma unroll
    for (int j = 0; j < PMAX; ++j)
      if (j < p) {
        const T* ev = a.in + (j + 1) * a.P;
        lap_vec_z<T, V>(ev, m[j + 1], c[j + 1], n[j + 1], row, q.x0, zoff + q.ymr, zoff + q.ypr, a, l);
#pragma unroll
        for (int e = 0; e < V; ++e) o[e] = c[j + 1].v[e] - a.dtL * (ge[j][e] - a.ke * l[e]);
        st_vec_nt<T, V>(a.out + (j + 1) * a.P + i0, o);
      }
#pragma unroll
    for (int f = 0; f <= PMAX; ++f) {
      m[f] = c[f];
      c[f] = n[f];
    }
  }
}

template <typename T, int V>
__global__ void __launch_bounds__(256) fd_c_z_kernel(FdArgs<T> a, int zb) {
  ZCol q;
  if (!zcol<T, V>(a, zb, q)) return;
  FdVec<T, V> m = ld_vec<T, V>(a.mu + (long long)((q.z0 - 1) & (a.nz - 1)) * q.plane + q.rest);
  FdVec<T, V> c = ld_vec<T, V>(a.mu + (long long)q.z0 * q.plane + q.rest);
  for (int k = 0; k < zb; ++k) {
    const int z = q.z0 + k;
    const long long zoff = (long long)z * q.plane;
    const long long i0 = zoff + q.rest;
    const FdVec<T, V> n = ld_vec<T, V>(a.mu + (long long)((z + 1) & (a.nz - 1)) * q.plane + q.rest);
    const FdVec<T, V> cu = ld_vec<T, V>(a.in + i0);
    T l[V], o[V];
    lap_vec_z<T, V>(a.mu, m, c, n, zoff + (q.rest - q.x0), q.x0, zoff + q.ymr, zoff + q.ypr, a, l);
#pragma unroll
    for (int e = 0; e < V; ++e) o[e] = cu.v[e] + a.dtM * l[e];
    st_vec_nt<T, V>(a.out + i0, o);
    m = c;
    c = n;
  }
}

// Marching kernels with the current plane staged in LDS.  A work-group of
// FD_ZL_WG threads owns a tile of R = FD_ZL_WG V / nx consecutive y rows
// (one vector per thread) of one block of planes; per plane it writes its
// centre vectors (kept in registers from the previous plane, as above) and
// the two halo rows y0 - 1 and y0 + R of every field it differentiates into
// LDS, and takes the y and x neighbours from there.  Each field is then
// read about (R + 2) / R times per step instead of once per neighbour row.
// Same arithmetic, in the same order, as the other FD step kernels.
constexpr int FD_ZL_WG = 512;

template <typename T, int V>
__device__ __forceinline__ void lap_lds(const T* __restrict__ tile, int r, int x0, int nx,
                                        const FdVec<T, V>& zm, const FdVec<T, V>& cv,
                                        const FdVec<T, V>& zp, const FdArgs<T>& a, T* out) {
  // tile rows: 0 = y0 - 1, 1..R = own rows, R + 1 = y0 + R
  const T* up = tile + (long long)r * nx;        // row y - 1
  const T* dn = tile + (long long)(r + 2) * nx;  // row y + 1
  const T* me = tile + (long long)(r + 1) * nx;
  const FdVec<T, V> vm = *reinterpret_cast<const FdVec<T, V>*>(up + x0);
  const FdVec<T, V> vp = *reinterpret_cast<const FdVec<T, V>*>(dn + x0);
  const T xl = me[(x0 - 1) & (nx - 1)], xr = me[(x0 + V) & (nx - 1)];
#pragma unroll
  for (int k = 0; k < V; ++k) {
    const T c = cv.v[k];
    const T left = k == 0 ? xl : cv.v[k - 1];
    const T right = k == V - 1 ? xr : cv.v[k + 1];
    T rr = (right - T(2) * c + left) * a.ix2 + (vp.v[k] - T(2) * c + vm.v[k]) * a.iy2;
    rr += (zp.v[k] - T(2) * c + zm.v[k]) * a.iz2;
    out[k] = rr;
  }
}

// Tile of this work-group: first row y0, first plane z0, and this thread's
// row r within the tile and x0.  Blocks are mapped to XCD-contiguous eighths
// of the grid as in zcol, so neighbouring tiles share an L2.
struct ZTile {
  long long plane;
  int y0, z0, r, x0, R;
};

template <typename T, int V>
__device__ __forceinline__ bool ztile(const FdArgs<T>& a, int zb, ZTile& q) {
  const int tpr = a.nx / V;  // threads per row
  q.R = FD_ZL_WG / tpr;
  const int tiles = a.ny / q.R;
  const unsigned b = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  if ((long long)b >= (long long)tiles * (a.nz / zb)) return false;
  q.y0 = int(b % tiles) * q.R;
  q.z0 = int(b / tiles) * zb;
  q.r = threadIdx.x / tpr;
  q.x0 = int(threadIdx.x - q.r * tpr) * V;
  q.plane = (long long)a.nx * a.ny;
  return true;
}

// Stage plane z of `nf` fields (field stride fs from base) into LDS: the
// centre vectors from registers, the halo rows from memory (threads of the
// first two rows of the tile load them).
template <typename T, int V, int NF>
__device__ __forceinline__ void stage_plane(T* lds, const T* __restrict__ base, long long fs,
                                            const FdVec<T, V>* cv, int nf, int z,
                                            const ZTile& q, const FdArgs<T>& a) {
  const int tsz = (q.R + 2) * a.nx;  // LDS values per field
#pragma unroll
  for (int f = 0; f < NF; ++f)
    if (f < nf)
      *reinterpret_cast<FdVec<T, V>*>(lds + f * tsz + (q.r + 1) * a.nx + q.x0) = cv[f];
  if (q.r < 2) {
    const int yh = q.r == 0 ? ((q.y0 - 1) & (a.ny - 1)) : ((q.y0 + q.R) & (a.ny - 1));
    const int lr = q.r == 0 ? 0 : q.R + 1;
    const long long off = (long long)z * q.plane + (long long)yh * a.nx + q.x0;
#pragma unroll
    for (int f = 0; f < NF; ++f)
      if (f < nf)
        *reinterpret_cast<FdVec<T, V>*>(lds + f * tsz + lr * a.nx + q.x0) =
            ld_vec<T, V>(base + f * fs + off);
  }
}

template <typename T, int PMAX, int V, bool FIXF = false>
__global__ void __launch_bounds__(FD_ZL_WG) fd_mu_zl_kernel(FdArgs<T> a, int zb) {
  extern __shared__ __align__(16) unsigned char fd_lds_raw[];
  T* lds = reinterpret_cast<T*>(fd_lds_raw);
  ZTile q;
  if (!ztile<T, V>(a, zb, q)) return;
  const int p = FIXF ? PMAX : a.F - 1;
  const int tsz = (q.R + 2) * a.nx;
  const long long rest = (long long)(q.y0 + q.r) * a.nx + q.x0;
  FdVec<T, V> m[PMAX + 1], c[PMAX + 1], n[PMAX + 1];
  const long long zm0 = (long long)((q.z0 - 1) & (a.nz - 1)) * q.plane + rest;
  const long long zc0 = (long long)q.z0 * q.plane + rest;
#pragma unroll
  for (int f = 0; f <= PMAX; ++f)
    if (f <= p) {
      m[f] = ld_vec<T, V>(a.in + f * a.P + zm0);
      c[f] = ld_vec<T, V>(a.in + f * a.P + zc0);
    }
  for (int k = 0; k < zb; ++k) {
    const int z = q.z0 + k;
    const long long i0 = (long long)z * q.plane + rest;
    const long long zn = (long long)((z + 1) & (a.nz - 1)) * q.plane + rest;
#pragma unroll
    for (int f = 0; f <= PMAX; ++f)
      if (f <= p) n[f] = ld_vec<T, V>(a.in + f * a.P + zn);
    stage_plane<T, V, PMAX + 1>(lds, a.in, a.P, c, p + 1, z, q, a);
    __syncthreads();
    T gc[V], ge[PMAX][V];
#pragma unroll
    for (int e = 0; e < V; ++e) {
      T eta[PMAX], g[PMAX];
#pragma unroll
      for (int j = 0; j < PMAX; ++j) {
        eta[j] = (j < p) ? c[j + 1].v[e] : T(0);
        g[j] = T(0);
      }
      fe_grad<T, PMAX>(a.fe, p, c[0].v[e], eta, gc[e], g);
#pragma unroll
      for (int j = 0; j < PMAX; ++j) ge[j][e] = g[j];
    }
    T l[V], o[V];
    lap_lds<T, V>(lds, q.r, q.x0, a.nx, m[0], c[0], n[0], a, l);
#pragma unroll
    for (int e = 0; e < V; ++e) o[e] = gc[e] - a.kc * l[e];
    st_vec_nt<T, V>(a.mu + i0, o);
#pragma unroll
    for (int j = 0; j < PMAX; ++j)
      if (j < p) {
        lap_lds<T, V>(lds + (j + 1) * tsz, q.r, q.x0, a.nx, m[j + 1], c[j + 1], n[j + 1], a, l);
#pragma unroll
        for (int e = 0; e < V; ++e) o[e] = c[j + 1].v[e] - a.dtL * (ge[j][e] - a.ke * l[e]);
        st_vec_nt<T, V>(a.out + (j + 1) * a.P + i0, o);
      }
    __syncthreads();
#pragma unroll
    for (int f = 0; f <= PMAX; ++f) {
      m[f] = c[f];
      c[f] = n[f];
    }
  }
}

template <typename T, int V>
__global__ void __launch_bounds__(FD_ZL_WG) fd_c_zl_kernel(FdArgs<T> a, int zb) {
  extern __shared__ __align__(16) unsigned char fd_lds_raw[];
  T* lds = reinterpret_cast<T*>(fd_lds_raw);
  ZTile q;
  if (!ztile<T, V>(a, zb, q)) return;
  const long long rest = (long long)(q.y0 + q.r) * a.nx + q.x0;
  FdVec<T, V> m = ld_vec<T, V>(a.mu + (long long)((q.z0 - 1) & (a.nz - 1)) * q.plane + rest);
  FdVec<T, V> c = ld_vec<T, V>(a.mu + (long long)q.z0 * q.plane + rest);
  for (int k = 0; k < zb; ++k) {
    const int z = q.z0 + k;
    const long long i0 = (long long)z * q.plane + rest;
    const FdVec<T, V> n = ld_vec<T, V>(a.mu + (long long)((z + 1) & (a.nz - 1)) * q.plane + rest);
    const FdVec<T, V> cu = ld_vec<T, V>(a.in + i0);
    stage_plane<T, V, 1>(lds, a.mu, 0, &c, 1, z, q, a);
    __syncthreads();
    T l[V], o[V];
    lap_lds<T, V>(lds, q.r, q.x0, a.nx, m, c, n, a, l);
#pragma unroll
    for (int e = 0; e < V; ++e) o[e] = cu.v[e] + a.dtM * l[e];
    st_vec_nt<T, V>(a.out + i0, o);
    __syncthreads();
    m = c;
    c = n;
  }
}

// Laplacian with the y neighbours one row up and down in an LDS tile (`me`:
// this thread's row, row pitch nx) and the z neighbours in registers.
template <typename T, int V>
__device__ __forceinline__ void fd_lap_rows(const T* __restrict__ me, int nx, int x0, int xm, int xp,
                                            const FdVec<T, V>& zm, const FdVec<T, V>& cv,
                                            const FdVec<T, V>& zp, const FdArgs<T>& a, T* out) {
  const FdVec<T, V> vm = *reinterpret_cast<const FdVec<T, V>*>(me - nx + x0);
  const FdVec<T, V> vp = *reinterpret_cast<const FdVec<T, V>*>(me + nx + x0);
  const T xl = me[xm], xr = me[xp];
#pragma unroll
  for (int k = 0; k < V; ++k) {
    const T c = cv.v[k];
    const T left = k == 0 ? xl : cv.v[k - 1];
    const T right = k == V - 1 ? xr : cv.v[k + 1];
    T r = (right - T(2) * c + left) * a.ix2 + (vp.v[k] - T(2) * c + vm.v[k]) * a.iy2;
    r += (zp.v[k] - T(2) * c + zm.v[k]) * a.iz2;
    out[k] = r;
  }
}

// ---------------------------------------------------------------------------
// Fused step: mu stays on the chip.  A work-group owns a tile of rows and
// computes mu on them and on the halo the Laplacian of mu reads, so one
// launch reads the F fields and writes the F fields (2F instead of 2F + 3
// arrays through memory, and one launch instead of two).
//
// Points in 2D and in the marching form: thread row rr = 0 .. T - 1 of a tile
// holds grid row y0 - 1 + rr; rows 1 .. T - 2 are the tile's own, the first
// and last only supply mu.  Every thread takes V consecutive x points.

// mu at one point of a 2D grid (the tile's left and right edge columns).
template <typename T, int P>
__device__ __forceinline__ T fd_mu_point(const FdArgs<T>& a, int x, int y) {
  const T* c = a.in;
  const long long row = (long long)y * a.nx;
  const T cc = c[row + x];
  const T xl = c[row + ((x - 1) & (a.nx - 1))], xr = c[row + ((x + 1) & (a.nx - 1))];
  const T ym = c[(long long)((y - 1) & (a.ny - 1)) * a.nx + x];
  const T yp = c[(long long)((y + 1) & (a.ny - 1)) * a.nx + x];
  T eta[P], ge[P], gc;
#pragma unroll
  for (int j = 0; j < P; ++j) eta[j] = a.in[(j + 1) * a.P + row + x];
  fe_grad<T, P, -1, P>(a.fe, P, cc, eta, gc, ge);
  const T l = (xr - T(2) * cc + xl) * a.ix2 + (yp - T(2) * cc + ym) * a.iy2;
  return gc - a.kc * l;
}

// 2D.  The tile is FD2_LANES vectors wide (or the whole row if that is
// shorter) and FD2_ROWS - 2 rows high.  The neighbours of the fields come
// from the caches as in fd_mu_kernel; mu goes through LDS, whose two columns
// beyond the tile's edges are filled by lanes of the two halo rows (which
// have no order parameters to advance).
constexpr int FD2_ROWS = 8;
constexpr int FD2_LANES = 64;  // threads per row of a tile

template <typename T, int P, int V>
__global__ void __launch_bounds__(FD2_ROWS * FD2_LANES) fd2_fused_kernel(FdArgs<T> a, int lanes, int xtiles, int ntiles) {
  constexpr int PITCH = FD2_LANES * V + 2 * V;  // columns -1 .. 64 V at offset V
  __shared__ __align__(16) T mu[FD2_ROWS * PITCH];
  const unsigned b = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);  // contiguous band per XCD
  if (int(b) >= ntiles) return;
  const int yt = int(b) / xtiles;
  const int xt = int(b) - yt * xtiles;
  const int rr = int(threadIdx.x) / lanes;
  const int lane = int(threadIdx.x) - rr * lanes;
  const int y0 = yt * (FD2_ROWS - 2);
  const int y = (y0 - 1 + rr) & (a.ny - 1);
  const int xl0 = lane * V;                 // x within the tile
  const int x0 = xt * lanes * V + xl0;
  const bool own = rr >= 1 && rr <= FD2_ROWS - 2 && y0 - 1 + rr < a.ny;
  const long long i0 = (long long)y * a.nx + x0;
  NbV n;
  n.ym = (long long)((y - 1) & (a.ny - 1)) * a.nx + x0;
  n.yp = (long long)((y + 1) & (a.ny - 1)) * a.nx + x0;
  n.xl = i0 - x0 + ((x0 - 1) & (a.nx - 1));
  n.xr = i0 - x0 + ((x0 + V) & (a.nx - 1));
  n.zm = n.zp = i0;
  T* mrow = mu + rr * PITCH + V;

  const FdVec<T, V> cc = ld_vec<T, V>(a.in + i0);
  FdVec<T, V> ce[P];
#pragma unroll
  for (int j = 0; j < P; ++j) ce[j] = ld_vec<T, V>(a.in + (j + 1) * a.P + i0);
  T l[V], m[V], gc[V], ge[P][V];
  lap_vec2<T, V>(a.in, cc, n, a, l);
#pragma unroll
  for (int k = 0; k < V; ++k) {
    T eta[P], g[P];
#pragma unroll
    for (int j = 0; j < P; ++j) eta[j] = ce[j].v[k];
    fe_grad<T, P, -1, P>(a.fe, P, cc.v[k], eta, gc[k], g);
#pragma unroll
    for (int j = 0; j < P; ++j) ge[j][k] = g[j];
    m[k] = gc[k] - a.kc * l[k];
  }
  st_vec<T, V>(mrow + xl0, m);
  if (xtiles > 1) {
    // edge columns: row 0's lanes the left ones, the last row's the right
    const int e = lane + 1;  // thread row whose edge this lane fills
    if (e <= FD2_ROWS - 2) {
      const int ye = (y0 - 1 + e) & (a.ny - 1);
      const int xb = xt * lanes * V;
      if (rr == 0) mu[e * PITCH + V - 1] = fd_mu_point<T, P>(a, (xb - 1) & (a.nx - 1), ye);
      if (rr == FD2_ROWS - 1) mu[e * PITCH + V + lanes * V] = fd_mu_point<T, P>(a, (xb + lanes * V) & (a.nx - 1), ye);
    }
  }
  if (own) {
    T o[V];
#pragma unroll
    for (int j = 0; j < P; ++j) {
      lap_vec2<T, V>(a.in + (j + 1) * a.P, ce[j], n, a, l);
#pragma unroll
      for (int k = 0; k < V; ++k) o[k] = ce[j].v[k] - a.dtL * (ge[j][k] - a.ke * l[k]);
      st_vec<T, V>(a.out + (j + 1) * a.P + i0, o);
    }
  }
  __syncthreads();
  if (own) {
    const FdVec<T, V> um = *reinterpret_cast<const FdVec<T, V>*>(mrow - PITCH + xl0);
    const FdVec<T, V> up = *reinterpret_cast<const FdVec<T, V>*>(mrow + PITCH + xl0);
    const int w = lanes * V;
    const T xl = xtiles > 1 ? mrow[xl0 - 1] : mrow[(xl0 - 1) & (w - 1)];
    const T xr = xtiles > 1 ? mrow[xl0 + V] : mrow[(xl0 + V) & (w - 1)];
    T o[V];
#pragma unroll
    for (int k = 0; k < V; ++k) {
      const T left = k == 0 ? xl : m[k - 1];
      const T right = k == V - 1 ? xr : m[k + 1];
      const T lm = (right - T(2) * m[k] + left) * a.ix2 + (up.v[k] - T(2) * m[k] + um.v[k]) * a.iy2;
      o[k] = cc.v[k] + a.dtM * lm;
    }
    st_vec<T, V>(a.out + i0, o);
  }
}

// 3D, large grids.  A work-group of WG threads owns all x of R = rows - 2 grid
// rows and marches over zb planes, with the planes q - 1, q, q + 1 of every
// field (PREF: also q + 2, loaded an iteration ahead) and mu of q - 2, q - 1, q
// in registers; plane q of the fields (one halo row on each side, two for c)
// and the planes q - 1 and q of mu are in LDS for the y and x neighbours.
// Iteration q advances eta of plane q and c of plane q - 1.  Bound by memory:
// 256^3, F = 5, FP32 138 us per step (671 MB read and written once, 4.9 TB/s)
// against 176 us of the two kernels (872 MB); FP64 244 against 392 us.
template <typename T, int P, int V, int WG, bool PREF>
__global__ void __launch_bounds__(WG) fd3_march_kernel(FdArgs<T> a, int zb, int rows, int ntiles) {
  extern __shared__ __align__(16) unsigned char fd_lds_raw[];
  const int nx = a.nx;
  const int tpr = nx / V;
  T* lc = reinterpret_cast<T*>(fd_lds_raw);  // c: thread rows -1 .. rows
  T* le = lc + (rows + 2) * nx;              // eta_j: thread rows 0 .. rows - 1 each
  T* lm = le + P * rows * nx;                // mu: two planes of the same
  const unsigned b = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);  // contiguous eighth per XCD
  const int R = rows - 2;
  const int ytiles = (a.ny + R - 1) / R;
  if (int(b) >= ntiles) return;  // work-group uniform
  const int zt = int(b) / ytiles;
  const int z0 = zt * zb;
  const int y0 = (int(b) - zt * ytiles) * R;
  const int rr = int(threadIdx.x) / tpr;
  const int x0 = (int(threadIdx.x) - rr * tpr) * V;
  const int y = (y0 - 1 + rr) & (a.ny - 1);
  const bool own = rr >= 1 && rr <= R && y0 - 1 + rr < a.ny;
  const bool top = rr == 0, bot = rr == rows - 1;
  const long long plane = (long long)nx * a.ny;
  const long long rest = (long long)y * nx + x0;
  const long long halo = (long long)((y + (top ? -1 : 1)) & (a.ny - 1)) * nx + x0;  // c row beyond the halo
  const int mz = a.nz - 1;
  const int xm = (x0 - 1) & (nx - 1), xp = (x0 + V) & (nx - 1);
  T* myc = lc + (rr + 1) * nx;
  T* mye = le + rr * nx;

  FdVec<T, V> m[P + 1], c[P + 1], n[P + 1], nn[P + 1];
  FdVec<T, V> hc;        // c of the row beyond the halo (first and last thread row)
  FdVec<T, V> mua, mub;  // mu of planes q - 2 and q - 1
#pragma unroll
  for (int k = 0; k < V; ++k) mua.v[k] = mub.v[k] = T(0);
  m[0] = ld_vec<T, V>(a.in + ((z0 - 2) & mz) * plane + rest);
#pragma unroll
  for (int f = 0; f <= P; ++f) c[f] = ld_vec<T, V>(a.in + f * a.P + ((z0 - 1) & mz) * plane + rest);
#pragma unroll
  for (int f = 1; f <= P; ++f) m[f] = c[f];  // (not used: eta of plane z0 - 1 is not advanced)
#pragma unroll
  for (int f = 0; f <= P; ++f) n[f] = ld_vec<T, V>(a.in + f * a.P + (z0 & mz) * plane + rest);
  hc = ld_vec<T, V>(a.in + ((z0 - 1) & mz) * plane + halo);
  for (int i = 0; i < zb + 2; ++i) {
    const int q = z0 - 1 + i;
    const long long zq = (q & mz) * plane;
    if (!PREF && i > 0) {
      const long long zn = ((q + 1) & mz) * plane + rest;
#pragma unroll
      for (int f = 0; f <= P; ++f) n[f] = ld_vec<T, V>(a.in + f * a.P + zn);
    }
    *reinterpret_cast<FdVec<T, V>*>(myc + x0) = c[0];
#pragma unroll
    for (int j = 0; j < P; ++j) *reinterpret_cast<FdVec<T, V>*>(mye + j * rows * nx + x0) = c[j + 1];
    if (top) *reinterpret_cast<FdVec<T, V>*>(myc - nx + x0) = hc;
    if (bot) *reinterpret_cast<FdVec<T, V>*>(myc + nx + x0) = hc;
    if (PREF) {
      const long long zn = ((q + 2) & mz) * plane + rest;
#pragma unroll
      for (int f = 0; f <= P; ++f) nn[f] = ld_vec<T, V>(a.in + f * a.P + zn);
    }
    if (top || bot) hc = ld_vec<T, V>(a.in + ((q + 1) & mz) * plane + halo);
    __syncthreads();
    T gc[V], ge[P][V];
#pragma unroll
    for (int k = 0; k < V; ++k) {
      T eta[P], g[P];
#pragma unroll
      for (int j = 0; j < P; ++j) eta[j] = c[j + 1].v[k];
      fe_grad<T, P, -1, P>(a.fe, P, c[0].v[k], eta, gc[k], g);
#pragma unroll
      for (int j = 0; j < P; ++j) ge[j][k] = g[j];
    }
    FdVec<T, V> mu;
    T l[V], o[V];
    fd_lap_rows<T, V>(myc, nx, x0, xm, xp, m[0], c[0], n[0], a, l);
#pragma unroll
    for (int k = 0; k < V; ++k) mu.v[k] = gc[k] - a.kc * l[k];
    T* lmq = lm + (i & 1) * rows * nx + rr * nx;
    *reinterpret_cast<FdVec<T, V>*>(lmq + x0) = mu;
    if (own && i >= 1 && i <= zb && q < a.nz) {
#pragma unroll
      for (int j = 0; j < P; ++j) {
        fd_lap_rows<T, V>(mye + j * rows * nx, nx, x0, xm, xp, m[j + 1], c[j + 1], n[j + 1], a, l);
#pragma unroll
        for (int k = 0; k < V; ++k) o[k] = c[j + 1].v[k] - a.dtL * (ge[j][k] - a.ke * l[k]);
        st_vec_nt<T, V>(a.out + (j + 1) * a.P + zq + rest, o);
      }
    }
    if (own && i >= 2 && q - 1 < a.nz) {
      // the other plane of mu, written in the iteration before
      fd_lap_rows<T, V>(lm + ((i + 1) & 1) * rows * nx + rr * nx, nx, x0, xm, xp, mua, mub, mu, a, l);
#pragma unroll
      for (int k = 0; k < V; ++k) o[k] = m[0].v[k] + a.dtM * l[k];
      st_vec_nt<T, V>(a.out + ((q - 1) & mz) * plane + rest, o);
    }
    __syncthreads();
    mua = mub;
    mub = mu;
#pragma unroll
    for (int f = 0; f <= P; ++f) {
      m[f] = c[f];
      c[f] = n[f];
      if (PREF) n[f] = nn[f];
    }
  }
}

// 3D, small grids with rows of at most 32 vectors: a tile of MY x MZ rows
// (all x) and the rows next to it in y and z, whose threads only supply mu.
// The fields' neighbours come from the caches as in fd_mu_kernel, mu goes
// through LDS.  One pass with one barrier: these grids are bound by latency
// and launches, so the mu of the halo rows computed twice costs less than a
// second kernel.
template <typename T, int P, int V, int MY, int MZ>
__global__ void __launch_bounds__(1024) fd3_tile_kernel(FdArgs<T> a, int ytiles, int ntiles) {
  constexpr int MM = MY * MZ;
  extern __shared__ __align__(16) unsigned char fd_lds_raw[];
  T* mu = reinterpret_cast<T*>(fd_lds_raw);  // [MM + 2 MY + 2 MZ][nx]
  const unsigned b = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);  // contiguous eighth per XCD
  if (int(b) >= ntiles) return;  // work-group uniform
  const int nx = a.nx;
  const int tpr = nx / V;
  const int zt = int(b) / ytiles;
  const int id = int(threadIdx.x) / tpr;
  const int x0 = (int(threadIdx.x) - id * tpr) * V;
  const bool own = id < MM;
  const int h = id - MM;
  int my, mz;
  if (own) {
    my = id % MY;
    mz = id / MY;
  } else if (h < 2 * MY) {
    my = h % MY;
    mz = h < MY ? -1 : MZ;
  } else {
    my = h < 2 * MY + MZ ? -1 : MY;
    mz = (h - 2 * MY) % MZ;
  }
  const int y = ((int(b) - zt * ytiles) * MY + my) & (a.ny - 1);
  const int z = (zt * MZ + mz) & (a.nz - 1);
  const long long i0 = ((long long)z * a.ny + y) * nx + x0;
  const NbV n = neighbours_vec<T, V>(a, i0);
  const FdVec<T, V> cc = ld_vec<T, V>(a.in + i0);
  FdVec<T, V> ce[P];
#pragma unroll
  for (int j = 0; j < P; ++j) ce[j] = ld_vec<T, V>(a.in + (j + 1) * a.P + i0);
  T l[V], o[V], m[V], ge[P][V];
  lap_vec3<T, V>(a.in, cc, n, a, l);
#pragma unroll
  for (int k = 0; k < V; ++k) {
    T eta[P], g[P], gc;
#pragma unroll
    for (int j = 0; j < P; ++j) eta[j] = ce[j].v[k];
    fe_grad<T, P, -1, P>(a.fe, P, cc.v[k], eta, gc, g);
#pragma unroll
    for (int j = 0; j < P; ++j) ge[j][k] = g[j];
    m[k] = gc - a.kc * l[k];
  }
  T* row = mu + id * nx;
  st_vec<T, V>(row + x0, m);
  if (own) {
#pragma unroll
    for (int j = 0; j < P; ++j) {
      lap_vec3<T, V>(a.in + (j + 1) * a.P, ce[j], n, a, l);
#pragma unroll
      for (int k = 0; k < V; ++k) o[k] = ce[j].v[k] - a.dtL * (ge[j][k] - a.ke * l[k]);
      st_vec<T, V>(a.out + (j + 1) * a.P + i0, o);
    }
  }
  __syncthreads();
  if (own) {
    const int ym = my > 0 ? id - 1 : MM + 2 * MY + mz;
    const int yp = my < MY - 1 ? id + 1 : MM + 2 * MY + MZ + mz;
    const int zm = mz > 0 ? id - MY : MM + my;
    const int zp = mz < MZ - 1 ? id + MY : MM + MY + my;
    const FdVec<T, V> um = ld_vec<T, V>(mu + ym * nx + x0), up = ld_vec<T, V>(mu + yp * nx + x0);
    const FdVec<T, V> wm = ld_vec<T, V>(mu + zm * nx + x0), wp = ld_vec<T, V>(mu + zp * nx + x0);
    const T xl = row[(x0 - 1) & (nx - 1)], xr = row[(x0 + V) & (nx - 1)];
#pragma unroll
    for (int k = 0; k < V; ++k) {
      const T left = k == 0 ? xl : m[k - 1];
      const T right = k == V - 1 ? xr : m[k + 1];
      T r = (right - T(2) * m[k] + left) * a.ix2 + (up.v[k] - T(2) * m[k] + um.v[k]) * a.iy2;
      r += (wp.v[k] - T(2) * m[k] + wm.v[k]) * a.iz2;
      o[k] = cc.v[k] + a.dtM * r;
    }
    st_vec<T, V>(a.out + i0, o);
  }
}

// partials[block] = {sum f(u), sum_d (dc/dx_d)^2, sum_i sum_d (deta_i/dx_d)^2, sum c}
// with forward differences, accumulated in double.  Each thread takes the V
// consecutive x points of one vector and adds them in increasing x.  Every
// value is loaded before any is used, so all loads are in flight together.
// Slots beyond F read field 0 again and are not used; in 2D the z neighbour
// vector is the centre one.
template <typename T, int PMAX, int V>
__global__ void __launch_bounds__(256) fd_energy_kernel(FdArgs<T> a) {
  __shared__ double red[4 * 4];
  const long long i0 = ((long long)blockIdx.x * blockDim.x + threadIdx.x) * V;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  if (i0 < a.P) {
    const NbV n = neighbours_vec<T, V>(a, i0);
    const int p = a.F - 1;
    constexpr int FM = PMAX + 1;
    FdVec<T, V> vc[FM], vy[FM], vz[FM];
    T vr[FM];
#pragma unroll
    for (int f = 0; f < FM; ++f) {
      const T* v = a.in + (long long)(f < a.F ? f : 0) * a.P;
      vc[f] = ld_vec<T, V>(v + i0);
      vy[f] = ld_vec<T, V>(v + n.yp);
      vz[f] = ld_vec<T, V>(v + n.zp);
      vr[f] = v[n.xr];
    }
#pragma unroll
    for (int k = 0; k < V; ++k) {
      T eta[PMAX];
#pragma unroll
      for (int j = 0; j < PMAX; ++j) eta[j] = (j < p) ? vc[j + 1].v[k] : T(0);
      acc[0] += fe_density<T, PMAX>(a.fe, p, vc[0].v[k], eta);
      acc[3] += double(vc[0].v[k]);
    }
#pragma unroll
    for (int f = 0; f < FM; ++f) {
      if (f < a.F) {
#pragma unroll
        for (int k = 0; k < V; ++k) {
          const double c = double(vc[f].v[k]);
          const double right = double(k == V - 1 ? vr[f] : vc[f].v[k + 1]);
          const double dx = (right - c) * a.ix;
          const double dy = (double(vy[f].v[k]) - c) * a.iy;
          double s = dx * dx + dy * dy;
          if (a.ndim == 3) {
            const double dz = (double(vz[f].v[k]) - c) * a.iz;
            s += dz * dz;
          }
          acc[f == 0 ? 1 : 2] += s;
        }
      }
    }
  }
  block_sum<4>(acc, red);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < 4; ++k) a.partials[4 * blockIdx.x + k] = acc[k];
  }
}

// Points per thread of the two step kernels: the widest vector (16 bytes at
// most) that still leaves 512 work-groups of 256 threads, so small grids
// keep enough waves in flight to hide load latency.
template <typename T>
static int fd_vec_width(long long P) {
  for (int v = 16 / int(sizeof(T)); v > 1; v /= 2)
    if (P / (256LL * v) >= 512) return v;
  return 1;
}

#ifndef PF_FD_ZLDS
#define PF_FD_ZLDS 1  // marching kernels with the current plane staged in LDS
#endif
#ifndef PF_FD_ZB
#define PF_FD_ZB 8  // planes per marching thread
#endif

// The two-kernel step (3D): XCD bands pay while the three neighbour planes of
// all F fields fit in half of one XCD's 4 MiB L2; beyond that the threads
// march along z.
template <typename T>
static int fd_bands(const FdArgs<T>& a) {
  return 3LL * a.F * a.nx * a.ny * (long long)sizeof(T) <= (2LL << 20) ? 1 : 0;
}

template <typename T, int PMAX, int V>
static int fd_go_v(int which, const FdArgs<T>& a, hipStream_t s) {
  const long long nv = a.P / V;  // nx >= 8 is a multiple of V
  const bool full = a.F == PMAX + 1;  // the mu kernel's p fixed at compile time
  if (!fd_bands(a)) {
    const int zb = a.nz < PF_FD_ZB ? a.nz : PF_FD_ZB;  // both powers of two
    // LDS-staged form: tiles of R >= 2 rows that divide Ny, with the plane
    // tiles of all F fields small enough for three work-groups per compute
    // unit (160 KiB of LDS); with fewer (FP64, F = 5, 256-point rows: two)
    // the register form was measured faster (3D 256^3 FD step 0.43 against
    // 0.39 ms)
    const int tpr = a.nx / V;
    const int R = tpr <= FD_ZL_WG ? FD_ZL_WG / tpr : 0;
    const size_t lds_mu = size_t(a.F) * (R + 2) * a.nx * sizeof(T);
    if (PF_FD_ZLDS && R >= 2 && R <= a.ny && lds_mu <= (160u << 10) / 3) {
      const long long nb = (long long)(a.ny / R) * (a.nz / zb);
      const int grid = int((nb + 7) / 8 * 8);
      if (which == 0 && full)
        hipLaunchKernelGGL((fd_mu_zl_kernel<T, PMAX, V, true>), dim3(grid), dim3(FD_ZL_WG), lds_mu, s, a, zb);
      else if (which == 0)
        hipLaunchKernelGGL((fd_mu_zl_kernel<T, PMAX, V>), dim3(grid), dim3(FD_ZL_WG), lds_mu, s, a, zb);
      else
        hipLaunchKernelGGL((fd_c_zl_kernel<T, V>), dim3(grid), dim3(FD_ZL_WG),
                           size_t(R + 2) * a.nx * sizeof(T), s, a, zb);
      return grid;
    }
    const int grid = int((nv / zb + 255) / 256 + 7) / 8 * 8;
    if (which == 0 && full) hipLaunchKernelGGL((fd_mu_z_kernel<T, PMAX, V, true>), dim3(grid), dim3(256), 0, s, a, zb);
    else if (which == 0) hipLaunchKernelGGL((fd_mu_z_kernel<T, PMAX, V>), dim3(grid), dim3(256), 0, s, a, zb);
    else hipLaunchKernelGGL((fd_c_z_kernel<T, V>), dim3(grid), dim3(256), 0, s, a, zb);
    return grid;
  }
  const int grid = int((nv + 255) / 256 + 7) / 8 * 8;
  if (which == 0 && full) hipLaunchKernelGGL((fd_mu_kernel<T, PMAX, V, true>), dim3(grid), dim3(256), 0, s, a);
  else if (which == 0) hipLaunchKernelGGL((fd_mu_kernel<T, PMAX, V>), dim3(grid), dim3(256), 0, s, a);
  else hipLaunchKernelGGL((fd_c_kernel<T, V>), dim3(grid), dim3(256), 0, s, a);
  return grid;
}

template <typename T, int P, int V>
static int fd2_fused(const FdArgs<T>& a, hipStream_t s) {
  const int tpr = a.nx / V;
  const int lanes = tpr < FD2_LANES ? tpr : FD2_LANES;
  const int xtiles = tpr / lanes;
  const int ntiles = xtiles * ((a.ny + FD2_ROWS - 3) / (FD2_ROWS - 2));
  const int grid = (ntiles + 7) / 8 * 8;
  hipLaunchKernelGGL((fd2_fused_kernel<T, P, V>), dim3(grid), dim3(FD2_ROWS * lanes), 0, s, a, lanes, xtiles, ntiles);
  return grid;
}

// The 3D step by tiles: MY x MZ rows per work-group.
template <typename T, int P, int V, int MY, int MZ>
static int fd3_tile_go(const FdArgs<T>& a, hipStream_t s) {
  const int ytiles = a.ny / MY;  // MY and MZ are powers of two of at most 8, like ny and nz at least
  const int ntiles = ytiles * (a.nz / MZ);
  const int rows = MY * MZ + 2 * MY + 2 * MZ;
  const int grid = (ntiles + 7) / 8 * 8;
  hipLaunchKernelGGL((fd3_tile_kernel<T, P, V, MY, MZ>), dim3(grid), dim3(rows * (a.nx / V)),
                     size_t(rows) * a.nx * sizeof(T), s, a, ytiles, ntiles);
  return grid;
}

// The 3D step by marching; 0 where a tile would have fewer than three rows of
// its own or does not fit LDS.
template <typename T, int P, int V, int WG, bool PREF>
static int fd3_march(const FdArgs<T>& a, hipStream_t s) {
  const int tpr = a.nx / V;
  int rows = WG / tpr;
  if (rows > a.ny + 2) rows = a.ny + 2;
  const size_t lds = (size_t(rows) * (P + 3) + 2) * a.nx * sizeof(T);
  if (rows < 5 || lds > (160u << 10)) return 0;
  const int R = rows - 2;
  const int ytiles = (a.ny + R - 1) / R;
  // as many z blocks as the chip has slots for work-groups, of 8 planes at least
  int nzb = 256 * (1024 / WG) / ytiles;
  if (nzb > a.nz / 8) nzb = a.nz / 8;
  if (nzb < 1) nzb = 1;
  const int zb = (a.nz + nzb - 1) / nzb;
  const int ntiles = ytiles * ((a.nz + zb - 1) / zb);
  const int grid = (ntiles + 7) / 8 * 8;
  hipLaunchKernelGGL((fd3_march_kernel<T, P, V, WG, PREF>), dim3(grid), dim3(rows * tpr), lds, s, a, zb, rows, ntiles);
  return grid;
}

// One step in one launch; 0 where the two-kernel step is taken.
// 2D: always fused (1024^2, F = 5, FP32 14.9 -> 11.8 us per step, 256^2 6.9 ->
// 3.6, 4096^2 220 -> 169; FP64 22.6 -> 19.4, 7.4 -> 4.3, 407 -> 309).
// 3D, from PF_FD3_MARCH_MB of fields (half of that with at most two order
// parameters, whose short steps the second launch costs more: 64 x 256 x 256, F = 3,
// FP32 31.8 -> 28.6 us; but F = 6, 32 x 256 x 256, 48 MB, FP32 29.3 -> 31.4): marching,
// in 512-lane work-groups with prefetch where a float row fits 64 lanes, else in
// 768-lane ones (256^3, F = 5, FP32 138 against 159 us; 512 x 256 x 256 has rows for
// the latter only).  Below that the marching work-groups are too few (128^3, F =
// 5, FP32 28.5 us against 25.9 of the two kernels).
// 3D, up to PF_FD3_TILE_MB of fields, or 128-point float rows with at most
// four order parameters below PF_FD3_MARCH_MB / 2: tiles (32^3, F = 5, FP32 7.4 ->
// 3.9 us, 64^3 9.3 -> 6.1, 128^3 25.9 -> 24.9; but 64 x 128^2, 21 MB: 16.3 -> 17.4, 128
// x 256 x 128, F = 5, FP32, 84 MB 46 -> 52; FP64 64^3 10.1 -> 7.4, 32 x 128^2, 21 MB: 15.1
// -> 17.7).  16- and 32-point rows go by one point per thread and leave the tiles
// a little earlier (FP32 32 x 256 x 128, F = 2, 8 MB 10.6 -> 11.9, 32 x 128^2, F = 3, 6
// MB 8.8 -> 7.9; FP64 32 x 64 x 128, F = 5, 10 MB 9.9 -> 10.5, F = 4, 8 MB 9.8 -> 9.1).
// 64-point double rows with more than five order parameters spill (64^3, p = 8:
// 14.2 -> 23.7 us) and stay with the two kernels.
#ifndef PF_FD3_MARCH_MB
#define PF_FD3_MARCH_MB 96
#endif
#ifndef PF_FD3_TILE_MB
#define PF_FD3_TILE_MB 11
#endif
template <typename T, int P>
static int fd_fused(const FdArgs<T>& a, hipStream_t s) {
  constexpr int VMAX = 16 / int(sizeof(T));
  if (a.ndim == 2) {
    const int v = fd_vec_width<T>(a.P);
    if constexpr (VMAX == 4) {
      if (v == 4) return fd2_fused<T, P, 4>(a, s);
    }
    return v == 2 ? fd2_fused<T, P, 2>(a, s) : fd2_fused<T, P, 1>(a, s);
  }
  constexpr int VM = P > 4 ? VMAX / 2 : VMAX;  // vectors that leave room in registers
  constexpr int words = (P + 1) * VM * int(sizeof(T)) / 4;
  const long long mb = ((long long)a.F * a.P * sizeof(T)) >> 20;
  if (mb >= (P <= 2 ? PF_FD3_MARCH_MB / 2 : PF_FD3_MARCH_MB)) {
    if constexpr (sizeof(T) == 4 && words > 12) {
      if (a.nx / VM <= 64) return fd3_march<T, P, VM, 512, true>(a, s);
    }
    return fd3_march<T, P, VM, 768, (words <= 12)>(a, s);
  }
  if constexpr (VMAX == 4 && P <= 4) {
    if (a.nx == 128 && mb < PF_FD3_MARCH_MB / 2) return fd3_tile_go<T, P, 4, 4, 4>(a, s);
  }
  const bool scalar_rows = a.nx == 16 || a.nx == 32;
  if (mb >= (scalar_rows ? (sizeof(T) == 4 ? PF_FD3_TILE_MB - 3 : PF_FD3_TILE_MB - 1) : PF_FD3_TILE_MB)) return 0;
  if (a.nx <= 8) return fd3_tile_go<T, P, 1, 8, 8>(a, s);   // 96 rows of 8 lanes
  if (a.nx <= 16) return fd3_tile_go<T, P, 1, 4, 8>(a, s);  // 56 of 16
  if (a.nx <= 32) return fd3_tile_go<T, P, 1, 4, 4>(a, s);  // 32 of 32
  if constexpr (sizeof(T) == 4 || P <= 5) {
    if (a.nx <= 64) return fd3_tile_go<T, P, 2, 4, 4>(a, s);
  }
  return 0;
}

template <typename T, int PMAX>
static int fd_go(int which, const FdArgs<T>& a, hipStream_t s) {
  if (which < 2) {
    const int v = fd_vec_width<T>(a.P);
    if constexpr (sizeof(T) == 4) {
      if (v == 4) return fd_go_v<T, PMAX, 4>(which, a, s);
    }
    if (v == 2) return fd_go_v<T, PMAX, 2>(which, a, s);
    return fd_go_v<T, PMAX, 1>(which, a, s);
  }
  // the energy pass: vectors as wide as the step kernels use
  const int v = fd_vec_width<T>(a.P);
  const int grid = int((a.P / v + 255) / 256);
  if constexpr (sizeof(T) == 4) {
    if (v == 4) {
      hipLaunchKernelGGL((fd_energy_kernel<T, PMAX, 4>), dim3(grid), dim3(256), 0, s, a);
      return grid;
    }
  }
  if (v == 2)
    hipLaunchKernelGGL((fd_energy_kernel<T, PMAX, 2>), dim3(grid), dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL((fd_energy_kernel<T, PMAX, 1>), dim3(grid), dim3(256), 0, s, a);
  return grid;
}

template <typename T>
static int fd_dispatch(int which, int p, const FdArgs<T>& a, hipStream_t s) {
  if (p <= 2) return fd_go<T, 2>(which, a, s);
  if (p <= 4) return fd_go<T, 4>(which, a, s);
  if (p <= 8) return fd_go<T, 8>(which, a, s);
  return -1;
}

template <typename T>
static int fd_fused_dispatch(int p, const FdArgs<T>& a, hipStream_t s) {
  switch (p) {
    case 1: return fd_fused<T, 1>(a, s);
    case 2: return fd_fused<T, 2>(a, s);
    case 3: return fd_fused<T, 3>(a, s);
    case 4: return fd_fused<T, 4>(a, s);
    case 5: return fd_fused<T, 5>(a, s);
    case 6: return fd_fused<T, 6>(a, s);
    case 7: return fd_fused<T, 7>(a, s);
    case 8: return fd_fused<T, 8>(a, s);
    default: return -1;
  }
}

template <>
int fd_fused_launch<float>(int p, const FdArgs<float>& a, hipStream_t s) {
  return fd_fused_dispatch<float>(p, a, s);
}
template <>
int fd_fused_launch<double>(int p, const FdArgs<double>& a, hipStream_t s) {
  return fd_fused_dispatch<double>(p, a, s);
}

template <>
int fd_launch<float>(int which, int p, const FdArgs<float>& a, hipStream_t s) {
  return fd_dispatch<float>(which, p, a, s);
}
template <>
int fd_launch<double>(int which, int p, const FdArgs<double>& a, hipStream_t s) {
  return fd_dispatch<double>(which, p, a, s);
}

}  // namespace pf
