// mhd_kernels.hpp -- stage kernels of the unsplit MHD update on a dense
// periodic level, and the diagnostics reductions.  Included once by
// mhd_api.hip, which instantiates and launches them.
//
// Storage (all SoA, x fastest, N = nx*ny*nz per component):
//   U [5][N]  rho, Mx, My, Mz, e at cell centres
//   B [3][N]  face-area-averaged field on the lower x/y/z face of each cell
//   W [8][N]  primitives rho, vx, vy, vz, p, Bcx, Bcy, Bcz (cell-centred field
//             = mean of the two opposite faces)
//   F [3][7][N] face fluxes of the lower face of each cell, per direction:
//             0 mass, 1..3 momentum x/y/z, 4 energy, 5 E_t1, 6 E_t2 -- the two
//             edge-parallel EMF components carried by the face (E = -V x B)
//   E [3][N]  edge EMFs: Ex on the x-edge at the lower (y, z) corner of the
//             cell, Ey at the lower (z, x) corner, Ez at the lower (x, y) corner.
//
// Work mapping: a launch covers units of cells -- the z-planes of a whole grid, its
// cells as one row, or the (edge + 2 halo)^3 item box of each listed group, with
// periodic wrap -- cut into blocks, a thread to a cell (mhd_layout.hpp).  Block ids
// are remapped so that each of the eight XCDs (which take blocks round-robin)
// works on a contiguous range of cells, which keeps stencil neighbours in that
// XCD's L2.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "mhd_device.hpp"
#include "mhd_layout.hpp"
#include "mhd_mlp.hpp"

namespace mhd {

constexpr int kBlock = 256;      // threads per block of the fixed-shape kernels

__device__ __forceinline__ long long lin(const Work& w, int i, int j, int k) {
  return ((long long)k * w.ny + j) * w.nx + i;
}

// neighbour index with periodic wrap; |di|, |dj|, |dk| <= grid size
__device__ __forceinline__ long long nbr(const Work& w, int i, int j, int k, int di, int dj, int dk) {
  return lin(w, wrapc(i + di, w.nx), wrapc(j + dj, w.ny), wrapc(k + dk, w.nz));
}

// Blocks are dispatched to the 8 XCDs round-robin (block b to XCD b % 8);
// the rank remaps them so each XCD gets a contiguous range of ranks.
__device__ __forceinline__ unsigned block_rank() {
  const unsigned nb = gridDim.x;
  const unsigned b = blockIdx.x;
  const unsigned q = nb >> 3;
  return b < (q << 3) ? (b & 7u) * q + (b >> 3) : b;
}

__device__ __forceinline__ long long block_linear_id() { return (long long)block_rank() * blockDim.x + threadIdx.x; }

// Persistent launches: a grid of at most a tuned number of blocks walks the
// work items with a grid-wide stride; the item count of a group list may be
// read from device memory, so a captured graph replays over a changed list.
__device__ __forceinline__ long long work_items(const Work& w) {
  if (w.n_dev) {
    long long n = (long long)*w.n_dev - w.gbase;
    n = n < 0 ? 0 : (n > w.gcount ? w.gcount : n);
    const long long m = (long long)w.box * w.box * w.box * n;
    return m < w.items ? m : w.items;
  }
  return w.items;
}
__device__ __forceinline__ long long item_stride() { return (long long)gridDim.x * blockDim.x; }

// cell of work item t.  (a, b, c) is the position inside the unit's box (the
// cell itself for a whole grid).  Item counts below 2^31 (all but whole levels of
// more cells) are split by multiplications (by_box, by_plane, by_row: item_divs).
__device__ __forceinline__ void cell_of(const Work& w, long long t, int& i, int& j, int& k, int& a, int& b, int& c) {
  const bool list = w.groups != nullptr;
  int g = 0;
  if (w.items < 1LL << 31) {
    unsigned l = (unsigned)t;
    const unsigned row = list ? w.box : w.nx, plane = row * (unsigned)(list ? w.box : w.ny);
    if (list) {
      g = (int)fdiv(w.by_box, l);
      l -= (unsigned)g * plane * (unsigned)w.box;
    }
    c = (int)fdiv(w.by_plane, l);
    l -= (unsigned)c * plane;
    b = (int)fdiv(w.by_row, l);
    a = (int)(l - (unsigned)b * row);
  } else {
    const long long row = list ? w.box : w.nx, plane = row * (list ? w.box : w.ny);
    if (list) {
      g = (int)(t / (plane * w.box));
      t -= g * plane * w.box;
    }
    c = (int)(t / plane);
    b = (int)((t - c * plane) / row);
    a = (int)(t - c * plane - b * row);
  }
  i = a; j = b; k = c;
  if (list) {
    const int* o = w.groups + 3LL * (w.gbase + g);
    i = wrapc((o[0] >> w.oshift) - w.halo + a, w.nx);
    j = wrapc((o[1] >> w.oshift) - w.halo + b, w.ny);
    k = wrapc((o[2] >> w.oshift) - w.halo + c, w.nz);
  }
}

__device__ __forceinline__ void cell_of(const Work& w, long long t, int& i, int& j, int& k) {
  int a, b, c;
  cell_of(w, t, i, j, k, a, b, c);
}

// loop over this thread's work items
#define FOR_ITEMS(w, t) for (long long t = block_linear_id(), t##_n = work_items(w); t < t##_n; t += item_stride())


// ---- addressing of the stage kernels
//
// A block covers part of one unit: one z-plane of a whole grid, or one listed
// group's item box.  The plane or box is then the same for the whole block, so
// its base address is scalar; a thread keeps one 32-bit byte offset inside it,
// and a neighbour costs nothing (a group box: every neighbour at a constant
// distance from the scalar base), one scalar address (a whole grid, along z)
// or one add of a wrapped distance (along x and y; kFlat: along z too).  The cell's coordinates
// come from two multiplications.  (One 64-bit linear index per thread, split
// by 64-bit divisions, and a 64-bit product per neighbour took 35-80 % of the
// stages' vector instructions.)  In a step a plane or box is below 4 GiB: planes of
// 2^29 cells would need more memory than the device has, since a level has at
// least four of them and at least 35 words of scratch per cell.  The kernels that
// need no scratch (CFL, diagnostics) take such a level by 64-bit level indices.
// A uniform address the compiler takes as it stands: without this it regroups
// (array + component + plane) + thread into (array + thread) + component and
// spends a 64-bit vector add per access instead of a scalar one (a tenth of
// the vector instructions of the reconstruction stage).
typedef __attribute__((address_space(1))) char gchar;   // device memory
__device__ __forceinline__ gchar* scalar(const void* p) {
  gchar* g = (gchar*)p;
  asm("" : "+s"(g));
  return g;
}
template <typename T>
__device__ __forceinline__ T load_at(gchar* base, unsigned off) {
  return *(__attribute__((address_space(1))) const T*)(base + off);
}
template <typename T>
__device__ __forceinline__ void store_at(gchar* base, unsigned off, T v) {
  *(__attribute__((address_space(1))) T*)(base + off) = v;
}

template <typename T, int L>
struct Cell {
  bool on;              // the thread has a cell
  int i, j, k;          // cell of the level
  int a, b, c;          // position in the group's item box (kList)
  unsigned o;           // byte offset in the plane or scratch box (kFlat: in the component)
  long long u;          // element offset of the plane or scratch box (uniform)
  long long p;          // level index (kList)

  __device__ __forceinline__ Cell(const Work& w, unsigned rank) {
    const unsigned unit = fdiv(w.by_chunks, rank);
    const unsigned l = (rank - unit * w.chunks) * blockDim.x + threadIdx.x;
    on = l < w.per;
    if (L == kList && w.groups == nullptr) {   // a whole grid by 64-bit level indices (read_mode)
      p = (long long)unit * w.per + l;
      on = on && p < w.N;
      const long long plane = (long long)w.nx * w.ny;
      k = (int)(p / plane);
      const long long r = p - k * plane;
      j = (int)(r / w.nx);
      i = (int)(r - (long long)j * w.nx);
      a = i; b = j; c = k;
      u = 0;
      o = 0;
    } else if constexpr (L == kList) {
      const unsigned box = w.box;
      c = (int)fdiv(w.by_plane, l);
      const unsigned r = l - (unsigned)c * box * box;
      b = (int)fdiv(w.by_row, r);
      a = (int)(r - (unsigned)b * box);
      const int g = w.gbase + (int)unit;
      const int* og = w.groups + 3LL * g;
      i = wrapc((og[0] >> w.oshift) - w.halo + a, w.nx);
      j = wrapc((og[1] >> w.oshift) - w.halo + b, w.ny);
      k = wrapc((og[2] >> w.oshift) - w.halo + c, w.nz);
      const long long sb = w.sb;
      u = (g + 1LL) * sb * sb * sb;
      o = (unsigned)(((c + w.soff) * w.sb + (b + w.soff)) * w.sb + (a + w.soff)) * (unsigned)sizeof(T);
      p = lin(w, i, j, k);
    } else if constexpr (L == kFlat) {
      flat(w, l);
    } else {
      j = (int)fdiv(w.by_row, l);
      i = (int)(l - (unsigned)j * (unsigned)w.nx);
      k = (int)unit;
      a = i; b = j; c = k;
      u = (long long)k * w.per;
      o = l * (unsigned)sizeof(T);
      p = 0;
    }
  }

  // (kFlat) the grid's cell l
  __device__ __forceinline__ void flat(const Work& w, unsigned l) {
    k = (int)fdiv(w.by_plane, l);
    const unsigned r = l - (unsigned)k * (unsigned)w.nx * (unsigned)w.ny;
    j = (int)fdiv(w.by_row, r);
    i = (int)(r - (unsigned)j * (unsigned)w.nx);
    a = i; b = j; c = k;
    u = 0;
    o = l * (unsigned)sizeof(T);
    p = 0;
  }
  struct AtCell {
    unsigned l;
  };
  __device__ __forceinline__ Cell(const Work& w, AtCell at) : on(true) { flat(w, at.l); }

  // The same cell with its offset taken anew: the compiler selects "scalar base
  // + 32-bit offset" addresses only where it sees the offset's extension in the
  // same basic block, so accesses behind a branch take a fresh copy.
  __device__ __forceinline__ Cell fresh() const {
    Cell r = *this;
    asm volatile("" : "+v"(r.o));
    return r;
  }

  // wrapped distances of the neighbours X cells along x and Y along y
  template <int X>
  __device__ __forceinline__ int dx(const Work& w) const {
    return X == 0 ? 0 : (X < 0 ? (i < -X ? X + w.nx : X) : (i >= w.nx - X ? X - w.nx : X));
  }
  template <int Y>
  __device__ __forceinline__ int dy(const Work& w) const {
    return Y == 0 ? 0 : (Y < 0 ? (j < -Y ? Y + w.ny : Y) : (j >= w.ny - Y ? Y - w.ny : Y));
  }
  // (kFlat) ... and Z along z
  template <int Z>
  __device__ __forceinline__ int dz(const Work& w) const {
    return Z == 0 ? 0 : (Z < 0 ? (k < -Z ? Z + w.nz : Z) : (k >= w.nz - Z ? Z - w.nz : Z));
  }
  // the scalar part of an address: component offset e, plane or box, and the
  // neighbour's share of it
  template <int X, int Y, int Z>
  __device__ __forceinline__ gchar* base(const Work& w, const T* arr, long long e) const {
    if constexpr (L == kList) e += u + X + (long long)Y * w.sb + (long long)Z * w.sb * w.sb;
    else if constexpr (Z == 0 || L == kFlat) e += u;
    else e += (long long)wrapc(k + Z, w.nz) * w.per;
    return scalar(arr + e);
  }
  template <int X, int Y, int Z>
  __device__ __forceinline__ unsigned off(const Work& w) const {
    unsigned v = o;   // distances wrap modulo 2^32, as the offset itself does
    if constexpr (L != kList && X != 0) v += (unsigned)dx<X>(w) * (unsigned)sizeof(T);
    if constexpr (L != kList && Y != 0) v += (unsigned)dy<Y>(w) * ((unsigned)w.nx * (unsigned)sizeof(T));
    if constexpr (L == kFlat && Z != 0) v += (unsigned)dz<Z>(w) * ((unsigned)w.nx * (unsigned)w.ny * (unsigned)sizeof(T));
    return v;
  }
  // one scratch component (arr + e) at the cell (X, Y, Z) away
  template <int X, int Y, int Z>
  __device__ __forceinline__ T at(const Work& w, const T* arr, long long e) const {
    return load_at<T>(base<X, Y, Z>(w, arr, e), off<X, Y, Z>(w));
  }
  // ... n cells along direction D
  template <int D, int n>
  __device__ __forceinline__ T along(const Work& w, const T* arr, long long e) const {
    return at<D == 0 ? n : 0, D == 1 ? n : 0, D == 2 ? n : 0>(w, arr, e);
  }
  __device__ __forceinline__ T here(const Work& w, const T* arr, long long e) const { return at<0, 0, 0>(w, arr, e); }
  __device__ __forceinline__ void put(const Work& w, T* arr, long long e, T v) const {
    store_at<T>(base<0, 0, 0>(w, arr, e), o, v);
  }
  // level index of the cell n along D (kList)
  template <int D, int n>
  __device__ __forceinline__ long long level_index(const Work& w) const {
    if constexpr (n == 0) return p;
    else if constexpr (D == 0) return p + dx<n>(w);
    else if constexpr (D == 1) return p + (long long)dy<n>(w) * w.nx;
    else return p + (long long)dz<n>(w) * w.nx * w.ny;
  }
  // one component of the level itself, n cells along D
  template <int D, int n>
  __device__ __forceinline__ T level(const Work& w, const T* arr, long long e) const {
    if constexpr (L == kList) return arr[e + level_index<D, n>(w)];
    else return along<D, n>(w, arr, e);
  }
  __device__ __forceinline__ void put_level(const Work& w, T* arr, long long e, T v) const {
    if constexpr (L == kList) arr[e + p] = v;
    else put(w, arr, e, v);
  }
  // the cell's level index (both modes)
  __device__ __forceinline__ long long index(const Work& w) const { return L == kList ? p : u + o / sizeof(T); }
};

// blocks of a stage: all units' chunks, the unit count of a group list read
// from device memory where the list lives there
template <int L>
__device__ __forceinline__ unsigned stage_blocks(const Work& w) {
  int n = w.units;
  if constexpr (L == kList) {
    if (w.n_dev) {
      const int m = *w.n_dev - w.gbase;
      n = m < 0 ? 0 : (m < n ? m : n);
    }
  }
  return (unsigned)n * w.chunks;
}

// loop over this block's chunks: c is the thread's cell (c.on: it has one)
#define FOR_CHUNKS(T, L, w, c)                                                           \
  for (unsigned c##_r = block_rank(), c##_n = stage_blocks<L>(w); c##_r < c##_n; c##_r += gridDim.x) \
    if (const Cell<T, L> c(w, w.rev ? c##_n - 1 - c##_r : c##_r); true)
#define FOR_CELLS(T, L, w, c) FOR_CHUNKS(T, L, w, c) if (c.on)

// time step source: explicit value or device scalar
struct DtSrc {
  double val;
  const double* ptr;
};

__device__ __forceinline__ double get_dt(const DtSrc& s) { return s.ptr ? *s.ptr : s.val; }

// CFL reduction of a context: the maximum signal speed (bit pattern of a
// positive double), the time step it gives, and the slots the blocks reduce
// into.  Thousands of blocks start together and all find their maximum larger
// than what is stored, so one shared slot would serialise their atomics (20-30
// us on 128^3, more than half of the primitive pass); 64 slots, each in a cache
// line of its own, divide that.  k_close_cfl takes their maximum and clears
// them for the next reduction.
constexpr int kCflSlots = 64, kCflPitch = 16;
struct Cfl {
  unsigned long long smax;
  double dt;
  unsigned long long pad[kCflPitch - 2];
  unsigned long long slot[kCflSlots * kCflPitch];
};

// ------------------------------------------------------------ reductions
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// ------------------------------------------------------------ primitives
// Energy storage of the mixed form: total energy in double, and the plasma
// beta below which the pressure is recovered in double.
struct Mix {
  double* E64;      // nullptr unless the mixed form
  double beta;
};

// gas pressure from the total energy (Eq. 5).  In the mixed form the
// subtraction p = (gam-1)(e - rho v^2/2 - B^2/2) is redone in double when
// the plasma beta 2p/|B|^2 of the float estimate is below mix.beta: there
// the kinetic and magnetic terms nearly cancel e.
template <typename T, bool MIX>
__device__ __forceinline__ T recover_pressure(double e, T d, T vx, T vy, T vz, T bx, T by, T bz, T gam,
                                              double beta) {
  const T b2 = bx * bx + by * by + bz * bz;
  const T pf = (gam - T(1)) * (T(e) - T(0.5) * d * (vx * vx + vy * vy + vz * vz) - T(0.5) * b2);
  if (MIX && T(2) * pf < T(beta) * b2) {
    const double dd = d, ux = vx, uy = vy, uz = vz, b2d = (double)bx * bx + (double)by * by + (double)bz * bz;
    return T(((double)gam - 1.0) * (e - 0.5 * dd * (ux * ux + uy * uy + uz * uz) - 0.5 * b2d));
  }
  return pf;
}

// primitives of a cell from its conserved values and its six faces (lower and
// upper of each direction)
template <typename T, bool MIX>
__device__ __forceinline__ void prims_from(T d, T mx, T my, T mz, T e, double e64, const T bl[3], const T bu[3], T gam,
                                           double beta, T out[8]) {
  const T bx = T(0.5) * (bl[0] + bu[0]);
  const T by = T(0.5) * (bl[1] + bu[1]);
  const T bz = T(0.5) * (bl[2] + bu[2]);
  const T id = T(1) / d;
  const T vx = mx * id, vy = my * id, vz = mz * id;
  T pr;
  if (MIX) {
    pr = recover_pressure<T, true>(e64, d, vx, vy, vz, bx, by, bz, gam, beta);
  } else {
    pr = (gam - T(1)) * (e - T(0.5) * d * (vx * vx + vy * vy + vz * vz) -
                         T(0.5) * (bx * bx + by * by + bz * bz));
  }
  out[0] = d; out[1] = vx; out[2] = vy; out[3] = vz; out[4] = pr; out[5] = bx; out[6] = by; out[7] = bz;
}

// primitives of a stage kernel's cell
template <typename T, bool MIX, int L>
__device__ __forceinline__ void cell_prims(const Work& w, const T* __restrict__ U, const T* __restrict__ B,
                                           const Mix& mix, const Cell<T, L>& c, T gam, T out[8]) {
  const long long N = w.N;
  const T bl[3] = {c.template level<0, 0>(w, B, 0), c.template level<0, 0>(w, B, N), c.template level<0, 0>(w, B, 2 * N)};
  const T bu[3] = {c.template level<0, 1>(w, B, 0), c.template level<1, 1>(w, B, N), c.template level<2, 1>(w, B, 2 * N)};
  T u[5];
#pragma unroll
  for (int m = 0; m < 5; ++m) u[m] = (MIX && m == 4) ? T(0) : c.template level<0, 0>(w, U, m * N);
  prims_from<T, MIX>(u[0], u[1], u[2], u[3], u[4], MIX ? mix.E64[c.index(w)] : 0.0, bl, bu, gam, mix.beta, out);
}

// component a of the cell's own EMF, -v x B, from its primitives
template <typename T>
__device__ __forceinline__ T cell_emf(const T q[8], int a) {
  const int b = (a + 1) % 3, c = (a + 2) % 3;
  return -(q[1 + b] * q[5 + c] - q[1 + c] * q[5 + b]);
}

// sum over directions of |v_d| + c_f,d, in double
template <typename T>
__device__ __forceinline__ double signal_speed(const T q[8], T gam) {
  double s = 0.0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int b = (a + 1) % 3, c = (a + 2) % 3;
    const T cf = fast_speed(q[0], q[4], q[5 + a], q[5 + b], q[5 + c], gam);
    s += (double)(dabs(q[1 + a]) + cf);
  }
  return s;
}

__device__ __forceinline__ void block_max_atomic(double v, Cfl* cfl) {
  __shared__ double red[kMaxBlock / 64];
  v = wave_max(v);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) red[wid] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    double m = red[0];
    for (int q = 1; q < (int)(blockDim.x >> 6); ++q) m = fmax(m, red[q]);
    // most blocks see a maximum already reached: skip their atomic
    unsigned long long* slot = cfl->slot + (blockIdx.x % kCflSlots) * kCflPitch;
    const unsigned long long bits = (unsigned long long)__double_as_longlong(m);
    if (m > 0.0 && bits > *(volatile unsigned long long*)slot) atomicMax(slot, bits);
  }
}

// Primitive state of every cell and the cell's EMF R = -v x B (three words that
// the edge EMFs read instead of v and B, six, which each of the twelve edges
// around a cell would multiply out again); optionally the CFL maximum signal
// speed and the sticky non-physical flag.
template <typename T, bool CFL, bool MIX, int L>
__global__ void __launch_bounds__(kMaxBlock) k_prim(Work w, const T* __restrict__ U, const T* __restrict__ B, Mix mix,
                                                 T* __restrict__ W, T* __restrict__ R, T gam, Cfl* cfl, int* flag) {
  double s = 0.0;
  FOR_CELLS(T, L, w, c) {
    T q[8];
    cell_prims<T, MIX, L>(w, U, B, mix, c, gam, q);
#pragma unroll
    for (int m = 0; m < 8; ++m) c.put(w, W, m * w.NS, q[m]);
#pragma unroll
    for (int m = 0; m < 3; ++m) c.put(w, R, m * w.NS, cell_emf(q, m));
    if (!(q[0] > T(0)) || !(q[4] > T(0))) atomicOr(flag, 1);
    else if (CFL) s = fmax(s, signal_speed(q, gam));
  }
  if (CFL) block_max_atomic(s, cfl);
}

// CFL maximum signal speed only
template <typename T, bool MIX, int L>
__global__ void __launch_bounds__(kBlock) k_cfl(Work w, const T* __restrict__ U, const T* __restrict__ B, Mix mix,
                                                T gam, Cfl* cfl, int* flag) {
  double s = 0.0;
  FOR_CELLS(T, L, w, c) {
    T q[8];
    cell_prims<T, MIX, L>(w, U, B, mix, c, gam, q);
    if (!(q[0] > T(0)) || !(q[4] > T(0))) atomicOr(flag, 1);
    else s = fmax(s, signal_speed(q, gam));
  }
  block_max_atomic(s, cfl);
}

// Close a CFL reduction (one wave): its maximum, dt = courant dx / smax, and
// optionally dt into an output scalar (or, with `least`, the smaller of the two),
// t += dt, and the maximum and the non-physical flag to pinned host memory.
__global__ void __launch_bounds__(kCflSlots) k_close_cfl(Cfl* cfl, double courant_dx, double* dt_out, double* t_out,
                                                         int least, const int* flag = nullptr, double* host = nullptr) {
  unsigned long long* slot = cfl->slot + threadIdx.x * kCflPitch;
  const double m = wave_max(__longlong_as_double((long long)*slot));
  *slot = 0ull;
  if (threadIdx.x) return;
  const double dt = courant_dx / m;
  cfl->smax = (unsigned long long)__double_as_longlong(m);
  cfl->dt = dt;
  if (dt_out && (!least || dt < *dt_out)) *dt_out = dt;
  if (t_out) *t_out += dt;
  if (host) {
    host[0] = m;
    host[1] = *flag ? 1.0 : 0.0;
  }
}

// ------------------------------------------------------------ fluxes
// 1D primitives of the cell n along D of a stage kernel's cell, in D's frame
template <typename T, int D, int n, int L>
__device__ __forceinline__ void load_frame(const Work& w, const T* __restrict__ W, const Cell<T, L>& c, T q[7]) {
  constexpr int t1 = (D + 1) % 3, t2 = (D + 2) % 3;
  constexpr int comp[7] = {0, 1 + D, 1 + t1, 1 + t2, 4, 5 + t1, 5 + t2};
#pragma unroll
  for (int m = 0; m < 7; ++m) q[m] = c.template along<D, n>(w, W, comp[m] * w.NS);
}

template <typename T, int D, int L>
__device__ __forceinline__ void store_flux(const Work& w, T* __restrict__ F, const Cell<T, L>& c0, const T f[7]) {
  const Cell<T, L> c = c0.fresh();
  constexpr int n = D, t1 = (D + 1) % 3, t2 = (D + 2) % 3;
  const long long NS = w.NS;
  constexpr int d = 7 * D;
  c.put(w, F, d * NS, f[0]);
  c.put(w, F, (d + 1 + n) * NS, f[1]);
  c.put(w, F, (d + 1 + t1) * NS, f[2]);
  c.put(w, F, (d + 1 + t2) * NS, f[3]);
  c.put(w, F, (d + 4) * NS, f[4]);
  c.put(w, F, (d + 5) * NS, f[6]);    // E_t1 = F_n[B_t2]
  c.put(w, F, (d + 6) * NS, -f[5]);   // E_t2 = -F_n[B_t1]
}

// RECON: 0 = first order (cell states), 1 = PLM with minmod on primitives,
// 2 = PPM (the limited parabolas' upper edge of the left cell and lower edge
// of the right cell, no tracing: the VL predictor centres the data in time).
// bn: the face's normal field.
template <typename T, int D, int RECON, int SOLVER, int L>
__device__ __forceinline__ int face_flux(const Work& w, const T* __restrict__ W, T bn, T* __restrict__ F,
                                         const Cell<T, L>& c0, T gam) {
  const Cell<T, L> c = c0.fresh();
  T wl[7], wr[7];
  load_frame<T, D, -1, L>(w, W, c, wl);
  load_frame<T, D, 0, L>(w, W, c, wr);
  if constexpr (RECON == 1) {
    T wll[7], wrr[7];
    load_frame<T, D, -2, L>(w, W, c, wll);
    load_frame<T, D, 1, L>(w, W, c, wrr);
#pragma unroll
    for (int m = 0; m < 7; ++m) {
      const T sL = minmod(wl[m] - wll[m], wr[m] - wl[m]);
      const T sR = minmod(wr[m] - wl[m], wrr[m] - wr[m]);
      wl[m] = wl[m] + T(0.5) * sL;
      wr[m] = wr[m] - T(0.5) * sR;
    }
  } else if constexpr (RECON == 2) {
    // cells -3, -2 and 1, 2 around the face (-1 and 0 are wl, wr)
    T q3[7], q2[7], p1[7], p2[7];
    load_frame<T, D, -3, L>(w, W, c, q3);
    load_frame<T, D, -2, L>(w, W, c, q2);
    load_frame<T, D, 1, L>(w, W, c, p1);
    load_frame<T, D, 2, L>(w, W, c, p2);
#pragma unroll
    for (int m = 0; m < 7; ++m) {
      T lo, hi, lo2, hi2;
      ppm_edges(q3[m], q2[m], wl[m], wr[m], p1[m], lo, hi);     // cell -1
      ppm_edges(q2[m], wl[m], wr[m], p1[m], p2[m], lo2, hi2);   // cell 0
      wl[m] = hi;
      wr[m] = lo2;
    }
  }
  T f[7];
  const int fb = riemann<SOLVER>(wl, wr, bn, gam, f);
  store_flux<T, D, L>(w, F, c, f);
  return fb;
}

__device__ __forceinline__ void block_count_atomic(int v, unsigned long long* counter) {
  __shared__ int red[kMaxBlock / 64];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) red[wid] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    int s = 0;
    for (int q = 0; q < (int)(blockDim.x >> 6); ++q) s += red[q];
    if (s) atomicAdd(counter, (unsigned long long)s);
  }
}

// One direction of the VL flux stage.  RECON 0 (predictor): the normal field is the
// level's B.  RECON 1 and 2 (corrector): it is the half-step scratch Bh, of which a
// direction reads its component at the own cell only and then overwrites it with that
// component of the cell's EMF of the half-step state, for the edge EMFs of the next
// stage.
template <typename T, int D, int RECON, int SOLVER, int L>
__device__ __forceinline__ int cell_flux(const Work& w, const T* __restrict__ W, const T* __restrict__ B, T* Bh,
                                         T* __restrict__ F, const Cell<T, L>& c, T gam) {
  const T bn = RECON == 0 ? c.template level<D, 0>(w, B, D * w.N) : c.here(w, (const T*)Bh, D * w.NS);
  if constexpr (RECON != 0) {
    constexpr int b = (D + 1) % 3, e = (D + 2) % 3;
    T q[8];
    q[1 + b] = c.here(w, W, (1 + b) * w.NS);
    q[1 + e] = c.here(w, W, (1 + e) * w.NS);
    q[5 + b] = c.here(w, W, (5 + b) * w.NS);
    q[5 + e] = c.here(w, W, (5 + e) * w.NS);
    c.put(w, Bh, D * w.NS, cell_emf(q, D));
  }
  return face_flux<T, D, RECON, SOLVER, L>(w, W, bn, F, c, gam);
}

// VL flux stage: all three directions of a cell, or one per launch row.
template <typename T, int RECON, int SOLVER, int L>
__global__ void __launch_bounds__(kMaxBlock) k_flux(Work w, const T* __restrict__ W, const T* __restrict__ B, T* Bh,
                                                 T* __restrict__ F, T gam, unsigned long long* nfb) {
  int fb = 0;
  FOR_CELLS(T, L, w, c) {
    if (gridDim.y == 1 || blockIdx.y == 0) fb += cell_flux<T, 0, RECON, SOLVER, L>(w, W, B, Bh, F, c, gam);
    if (gridDim.y == 1 || blockIdx.y == 1) fb += cell_flux<T, 1, RECON, SOLVER, L>(w, W, B, Bh, F, c, gam);
    if (gridDim.y == 1 || blockIdx.y == 2) fb += cell_flux<T, 2, RECON, SOLVER, L>(w, W, B, Bh, F, c, gam);
  }
  if (SOLVER == 0) block_count_atomic(fb, nfb);
}

// ------------------------------------------------------------ edge EMFs
template <typename T>
__device__ __forceinline__ T upwind(T m, T pos, T neg) {
  return m > T(0) ? pos : (m < T(0) ? neg : T(0.5) * (pos + neg));
}

// The upwind CT average of one edge from its four face EMFs (eb0, eb1 on the
// b-faces below and at the cell, ec0, ec1 on the c-faces), the faces' mass
// fluxes (mb*, mc*) and the reference EMFs of the four cells around the edge
// (r00 at the cell below in b and c, r10 below in c, r01 below in b, r11 the
// cell itself)
template <typename T>
__device__ __forceinline__ T edge_emf_core(T eb0, T eb1, T ec0, T ec1, T mb0, T mb1, T mc0, T mc1, T r00, T r10,
                                           T r01, T r11) {
  const T dc1 = upwind(mb1, r01 - ec0, r11 - ec1);
  const T dc0 = upwind(mb0, ec0 - r00, ec1 - r10);
  const T db1 = upwind(mc1, r10 - eb0, r11 - eb1);
  const T db0 = upwind(mc0, eb0 - r00, eb1 - r01);
  return T(0.25) * (eb0 + eb1 + ec0 + ec1) + T(0.25) * ((dc0 - dc1) + (db0 - db1));
}

// E_a on the edge at the lower (b, c) corner of a cell, (a, b, c) cyclic, from
// the four faces around the edge (upwind CT average of Gardiner & Stone 2005):
// each face value is extrapolated to the edge with the derivative taken in the
// upwind cell (sign of the face mass flux), and the four extrapolations are
// averaged.  R: the cells' own EMFs (cell_emf).
template <typename T, int A, int L>
__device__ __forceinline__ T edge_emf(const Work& w, const T* __restrict__ F, const T* __restrict__ R,
                                      const Cell<T, L>& p) {
  constexpr int b = (A + 1) % 3, c = (A + 2) % 3;
  constexpr int bx = b == 0 ? -1 : 0, by = b == 1 ? -1 : 0, bz = b == 2 ? -1 : 0;   // one cell down along b
  constexpr int cx = c == 0 ? -1 : 0, cy = c == 1 ? -1 : 0, cz = c == 2 ? -1 : 0;   // one cell down along c
  const long long N = w.NS;
  const long long fb = 7 * b * N, fc = 7 * c * N, ra = A * N;
  const T eb0 = p.template at<cx, cy, cz>(w, F, fb + 6 * N), eb1 = p.here(w, F, fb + 6 * N);
  const T ec0 = p.template at<bx, by, bz>(w, F, fc + 5 * N), ec1 = p.here(w, F, fc + 5 * N);
  const T mb0 = p.template at<cx, cy, cz>(w, F, fb), mb1 = p.here(w, F, fb);
  const T mc0 = p.template at<bx, by, bz>(w, F, fc), mc1 = p.here(w, F, fc);
  const T r00 = p.template at<bx + cx, by + cy, bz + cz>(w, R, ra), r10 = p.template at<cx, cy, cz>(w, R, ra);
  const T r01 = p.template at<bx, by, bz>(w, R, ra), r11 = p.here(w, R, ra);
  return edge_emf_core(eb0, eb1, ec0, ec1, mb0, mb1, mc0, mc1, r00, r10, r01, r11);
}

template <typename T, int L>
__global__ void __launch_bounds__(kMaxBlock) k_emf(Work w, const T* __restrict__ F, const T* __restrict__ R,
                                                T* __restrict__ E) {
  FOR_CELLS(T, L, w, c) {
    c.put(w, E, 0, edge_emf<T, 0, L>(w, F, R, c));
    c.put(w, E, w.NS, edge_emf<T, 1, L>(w, F, R, c));
    c.put(w, E, 2 * w.NS, edge_emf<T, 2, L>(w, F, R, c));
  }
}

// Edge EMFs of a whole grid on LDS tiles: each block stages, for its
// TX x TY x TZ cells and the layer below them along every direction, the
// cells' own EMFs R = -v x B (three components) and, per face direction,
// the face's mass flux and its two EMF components (twelve values per cell,
// each loaded once per tile instead of once per edge that uses it), then
// computes the three lower-corner edges of each of its cells from LDS with
// the arithmetic of k_emf.  Grids need not be multiples of the tile (cells
// past the grid idle; the staged layer wraps periodically: staged_coord).
template <typename T, int TX, int TY, int TZ>
__global__ void __launch_bounds__(TX * TY * TZ) k_emf_tiled(Work w, const T* __restrict__ F, const T* __restrict__ R,
                                                         T* __restrict__ E) {
  constexpr int HX = TX + 1, HY = TY + 1, HZ = TZ + 1, NH = HX * HY * HZ, NT = TX * TY * TZ;
  __shared__ T sR[3][NH];
  __shared__ T sF[3][3][NH];
  const int ntx = (w.nx + TX - 1) / TX, nty = (w.ny + TY - 1) / TY;
  const int tile = (int)(w.rev ? gridDim.x - 1 - block_rank() : block_rank());
  const int tx0 = (tile % ntx) * TX, ty0 = ((tile / ntx) % nty) * TY, tz0 = (tile / (ntx * nty)) * TZ;
  const long long N = w.NS;
  for (int h = threadIdx.x; h < NH; h += NT) {
    const int hx = h % HX, hy = (h / HX) % HY, hz = h / (HX * HY);
    const long long q = lin(w, staged_coord(tx0, hx, w.nx), staged_coord(ty0, hy, w.ny), staged_coord(tz0, hz, w.nz));
#pragma unroll
    for (int a = 0; a < 3; ++a) sR[a][h] = R[(long long)a * N + q];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      sF[d][0][h] = F[(long long)(7 * d) * N + q];
      sF[d][1][h] = F[(long long)(7 * d + 5) * N + q];
      sF[d][2][h] = F[(long long)(7 * d + 6) * N + q];
    }
  }
  __syncthreads();
  const int t = threadIdx.x;
  const int ax = t % TX, ay = (t / TX) % TY, az = t / (TX * TY);
  const int i = tx0 + ax, j = ty0 + ay, k = tz0 + az;
  if (i >= w.nx || j >= w.ny || k >= w.nz) return;
  const int h = ((az + 1) * HY + (ay + 1)) * HX + (ax + 1);
  const long long p = lin(w, i, j, k);
  constexpr int st[3] = {1, HX, HX * HY};
#pragma unroll
  for (int A = 0; A < 3; ++A) {
    const int b = (A + 1) % 3, c = (A + 2) % 3;
    const int hb = h - st[b], hc = h - st[c], hbc = h - st[b] - st[c];
    E[(long long)A * N + p] = edge_emf_core(sF[b][2][hc], sF[b][2][h], sF[c][1][hb], sF[c][1][h], sF[b][0][hc],
                                            sF[b][0][h], sF[c][0][hb], sF[c][0][h], sR[A][hbc], sR[A][hc],
                                            sR[A][hb], sR[A][h]);
  }
}

// ------------------------------------------------------------ updates
// U - r div F (Eq. 10), differences applied in the order x, y, z, for the first
// NM components.  In the mixed form the energy is updated in double from E64
// (returned in e64).
template <typename T, bool MIX, int L, int NM = 5>
__device__ __forceinline__ void cell_update(const Work& w, const T* U, const T* __restrict__ F, const Mix& mix,
                                            const Cell<T, L>& c, T r, T out[5], double& e64) {
  const long long N = w.N, NS = w.NS;
#pragma unroll
  for (int m = 0; m < NM; ++m) {
    const T xu = c.template along<0, 1>(w, F, m * NS), xl = c.here(w, F, m * NS);
    const T yu = c.template along<1, 1>(w, F, (7 + m) * NS), yl = c.here(w, F, (7 + m) * NS);
    const T zu = c.template along<2, 1>(w, F, (14 + m) * NS), zl = c.here(w, F, (14 + m) * NS);
    if (MIX && m == 4) {
      const double rd = (double)r;
      double v = mix.E64[c.index(w)];
      v -= rd * ((double)xu - (double)xl);
      v -= rd * ((double)yu - (double)yl);
      v -= rd * ((double)zu - (double)zl);
      e64 = v;
      out[4] = T(v);
      continue;
    }
    T v = c.template level<0, 0>(w, U, m * N);
    v -= r * (xu - xl);
    v -= r * (yu - yl);
    v -= r * (zu - zl);
    out[m] = v;
  }
  if (!MIX && NM == 5) e64 = (double)out[4];
}

// CT update (Eq. 13) of the lower A-face of the cell (n = 0) or of the next
// cell along A (n = 1)
template <typename T, int A, int n, int L>
__device__ __forceinline__ T face_update(const Work& w, const T* B, const T* __restrict__ E, const Cell<T, L>& p, T r) {
  constexpr int b = (A + 1) % 3, c = (A + 2) % 3;
  constexpr int X = A == 0 ? n : 0, Y = A == 1 ? n : 0, Z = A == 2 ? n : 0;
  const long long eb = b * w.NS, ec = c * w.NS;
  const T cu = p.template at<X + (b == 0), Y + (b == 1), Z + (b == 2)>(w, E, ec), cl = p.template at<X, Y, Z>(w, E, ec);
  const T bu = p.template at<X + (c == 0), Y + (c == 1), Z + (c == 2)>(w, E, eb), bl = p.template at<X, Y, Z>(w, E, eb);
  return p.template level<A, n>(w, B, A * w.N) - r * (cu - cl) + r * (bu - bl);
}

// Half step over dt/2: U^{n+1/2} and face B^{n+1/2} from the predictor fluxes
// and EMFs (cell-centred field from the updated faces, including the upper
// faces owned by the neighbours).  Writes Bh and, for VL, the primitives Wh;
// CTU's later stages need of the half-step cell state only its EMF (step 7),
// so there the energy is left out and three words R = -v x B replace Wh's
// eight.
template <typename T, bool MIX, bool CTU, int L>
__global__ void __launch_bounds__(kMaxBlock) k_half(Work w, const T* __restrict__ U, const T* __restrict__ B, Mix mix,
                                                 const T* __restrict__ F, const T* __restrict__ E, DtSrc dts,
                                                 T inv_dx, T gam, T* __restrict__ Wh, T* __restrict__ Bh) {
  const T r = T(0.5 * get_dt(dts)) * inv_dx;
  FOR_CELLS(T, L, w, c) {
    T u[5];
    double eh = 0.0;
    cell_update<T, MIX, L, CTU ? 4 : 5>(w, U, F, mix, c, r, u, eh);
    const T bl[3] = {face_update<T, 0, 0, L>(w, B, E, c, r), face_update<T, 1, 0, L>(w, B, E, c, r),
                     face_update<T, 2, 0, L>(w, B, E, c, r)};
    const T bu[3] = {face_update<T, 0, 1, L>(w, B, E, c, r), face_update<T, 1, 1, L>(w, B, E, c, r),
                     face_update<T, 2, 1, L>(w, B, E, c, r)};
    T q[8];
    if constexpr (CTU) {
      const T id = T(1) / u[0];
#pragma unroll
      for (int m = 0; m < 3; ++m) {
        q[1 + m] = u[1 + m] * id;
        q[5 + m] = T(0.5) * (bl[m] + bu[m]);
      }
#pragma unroll
      for (int m = 0; m < 3; ++m) c.put(w, Wh, m * w.NS, cell_emf(q, m));
    } else {
      prims_from<T, MIX>(u[0], u[1], u[2], u[3], u[4], eh, bl, bu, gam, mix.beta, q);
#pragma unroll
      for (int m = 0; m < 8; ++m) c.put(w, Wh, m * w.NS, q[m]);
    }
#pragma unroll
    for (int m = 0; m < 3; ++m) c.put(w, Bh, m * w.NS, bl[m]);
  }
}

// Full step over dt from time n (in place: each thread reads and writes only
// its own cell and its own lower faces).
//
// With a group list, a cell on the upper boundary of its group also updates
// the face it shares with the next cell when the next cell's group is not
// listed (occupancy map), so every face of a listed group advances exactly
// once and no face is read after another thread has written it.
template <typename T, bool MIX, int L>
__global__ void __launch_bounds__(kMaxBlock) k_final(Work w, T* __restrict__ U, T* __restrict__ B, Mix mix,
                                                  const T* __restrict__ F, const T* __restrict__ E, DtSrc dts,
                                                  T inv_dx) {
  const T r = T(get_dt(dts)) * inv_dx;
  const long long N = w.N;
  FOR_CELLS(T, L, w, c) {
    T u[5], bf[3];
    double e64;
    cell_update<T, MIX, L>(w, U, F, mix, c, r, u, e64);
    bf[0] = face_update<T, 0, 0, L>(w, B, E, c, r);
    bf[1] = face_update<T, 1, 0, L>(w, B, E, c, r);
    bf[2] = face_update<T, 2, 0, L>(w, B, E, c, r);
    T ux = T(0), uy = T(0), uz = T(0);
    bool ex = false, ey = false, ez = false;
    if constexpr (L == kList) {
      // the group's place in the occupancy map: its boundary cells look at the next one
      const auto listed = [&](int x, int y, int z) {
        return w.occ[((long long)wrapc(z, w.gnz) * w.gny + wrapc(y, w.gny)) * w.gnx + wrapc(x, w.gnx)] != 0;
      };
      const bool lx = c.a == w.edge - 1, ly = c.b == w.edge - 1, lz = c.c == w.edge - 1;
      if (lx || ly || lz) {
        const int gi = (int)fdiv(w.by_edge, c.i), gj = (int)fdiv(w.by_edge, c.j), gk = (int)fdiv(w.by_edge, c.k);
        ex = lx && !listed(gi + 1, gj, gk);
        ey = ly && !listed(gi, gj + 1, gk);
        ez = lz && !listed(gi, gj, gk + 1);
        if (ex) ux = face_update<T, 0, 1, L>(w, B, E, c, r);
        if (ey) uy = face_update<T, 1, 1, L>(w, B, E, c, r);
        if (ez) uz = face_update<T, 2, 1, L>(w, B, E, c, r);
      }
    }
#pragma unroll
    for (int m = 0; m < 5; ++m) c.put_level(w, U, m * N, u[m]);
    if (MIX) mix.E64[c.index(w)] = e64;
#pragma unroll
    for (int m = 0; m < 3; ++m) c.put_level(w, B, m * N, bf[m]);
    if constexpr (L == kList) {
      if (ex) B[c.template level_index<0, 1>(w)] = ux;
      if (ey) B[N + c.template level_index<1, 1>(w)] = uy;
      if (ez) B[2 * N + c.template level_index<2, 1>(w)] = uz;
    }
  }
}

// ------------------------------------------------------------ CTU
// Steps 1, 2, 5 and 6 are the face kernels of mhd_faces.hpp; here is step 5's
// correction of a state.

// Step 5's share of one cell, the same for the states at both its D-edges: dt/2
// times the transverse flux differences of step 2 (frame order: mass, normal
// and transverse momenta, energy) and the transverse part of -curl E from the
// step-3 EMFs E_D at the cell's four D-edges, averaged along the field's own
// axis to the two faces it is differenced between.
template <typename T>
struct Transverse {
  T g[5], c1, c2;
};

// Step 5: transverse correction of a state s of a cell on a face with normal
// field bn at time n and bnh after the half step.  The state enters conserved
// form with bn and leaves it with bnh (the transverse energy fluxes carry the
// normal field's change of magnetic energy).  The conserved transverse flux
// differences hold the div B terms of their directions, dBn/dn (0, B, v.B, v):
// momentum and energy get (dt/2)(B, v.B) dBn/dn, hd = (dt/2) times the cell's
// normal-field difference (the field's share is in the traced state).
// Non-physical results keep the input.
template <typename T>
__device__ __forceinline__ void correct_state(const Transverse<T>& tr, T bn, T bnh, T hd, T gam, T s[7]) {
  const T gm1 = gam - T(1), gm1inv = T(1) / gm1;
  const T vb = s[1] * bn + s[2] * s[5] + s[3] * s[6];
  const T d = s[0] - tr.g[0];
  const T mn = s[0] * s[1] + hd * bn - tr.g[1];
  const T m1 = s[0] * s[2] + hd * s[5] - tr.g[2];
  const T m2 = s[0] * s[3] + hd * s[6] - tr.g[3];
  const T e = s[4] * gm1inv + T(0.5) * s[0] * (s[1] * s[1] + s[2] * s[2] + s[3] * s[3]) +
              T(0.5) * (bn * bn + s[5] * s[5] + s[6] * s[6]) + hd * vb - tr.g[4];
  const T b1 = s[5] - tr.c1, b2 = s[6] + tr.c2;
  const T id = T(1) / d;
  const T vn = mn * id, v1 = m1 * id, v2 = m2 * id;
  const T p = gm1 * (e - T(0.5) * d * (vn * vn + v1 * v1 + v2 * v2) - T(0.5) * (bnh * bnh + b1 * b1 + b2 * b2));
  if (d > T(0) && p > T(0)) {
    s[0] = d; s[1] = vn; s[2] = v1; s[3] = v2; s[4] = p; s[5] = b1; s[6] = b2;
  }
}

// Step 5's share of the cell n along D
template <typename T, int D, int n, int L>
__device__ __forceinline__ Transverse<T> transverse_of(const Work& w, const T* __restrict__ F1,
                                                       const T* __restrict__ E1, const Cell<T, L>& c, T hr) {
  constexpr int t1 = (D + 1) % 3, t2 = (D + 2) % 3;
  constexpr int X = D == 0 ? n : 0, Y = D == 1 ? n : 0, Z = D == 2 ? n : 0;   // the source cell
  constexpr int comp[5] = {0, 1 + D, 1 + t1, 1 + t2, 4};
  const long long N = w.NS;
  Transverse<T> r;
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    const long long f1 = (7 * t1 + comp[m]) * N, f2 = (7 * t2 + comp[m]) * N;
    r.g[m] = hr * (c.template at<X + (t1 == 0), Y + (t1 == 1), Z + (t1 == 2)>(w, F1, f1) -
                   c.template at<X, Y, Z>(w, F1, f1)) +
             hr * (c.template at<X + (t2 == 0), Y + (t2 == 1), Z + (t2 == 2)>(w, F1, f2) -
                   c.template at<X, Y, Z>(w, F1, f2));
  }
  const long long ed = D * N;
  const T e00 = c.template at<X, Y, Z>(w, E1, ed);
  const T e10 = c.template at<X + (t1 == 0), Y + (t1 == 1), Z + (t1 == 2)>(w, E1, ed);
  const T e01 = c.template at<X + (t2 == 0), Y + (t2 == 1), Z + (t2 == 2)>(w, E1, ed);
  const T e11 =
      c.template at<X + (t1 == 0) + (t2 == 0), Y + (t1 == 1) + (t2 == 1), Z + (t1 == 2) + (t2 == 2)>(w, E1, ed);
  r.c1 = hr * (T(0.5) * (e01 + e11) - T(0.5) * (e00 + e10));
  r.c2 = hr * (T(0.5) * (e10 + e11) - T(0.5) * (e00 + e01));
  return r;
}

// the two states (wl, wr) of the cell's lower D-face corrected to the half-step
// normal field bnh
template <typename T, int D, int L>
__device__ __forceinline__ void correct_states(const Work& w, const T* __restrict__ F1, const T* __restrict__ E1,
                                               const T* __restrict__ B, T bnh, const Cell<T, L>& c, T hr, T gam,
                                               T wl[7], T wr[7]) {
  const T bn = c.template level<D, 0>(w, B, D * w.N);
  const T bn_lo = c.template level<D, -1>(w, B, D * w.N);
  const T bn_hi = c.template level<D, 1>(w, B, D * w.N);
  correct_state(transverse_of<T, D, -1, L>(w, F1, E1, c, hr), bn, bnh, hr * (bn - bn_lo), gam, wl);
  correct_state(transverse_of<T, D, 0, L>(w, F1, E1, c, hr), bn, bnh, hr * (bn_hi - bn), gam, wr);
}

// Occupancy map of a level's group list (list mode only) into occ[n]: cleared, then
// the listed groups marked.  One block does both where its passes over the map are
// few (two launches took 9.3 us, one 4.9 us on a map of 512, and a step of a
// hierarchy builds several); a larger map takes a launch for each.
__device__ __forceinline__ void occ_set(int* occ, const int* groups, int g, int edge, int gnx, int gny, int gnz) {
  const int gi = groups[3 * g] / edge, gj = groups[3 * g + 1] / edge, gk = groups[3 * g + 2] / edge;
  // origins outside the level are never written (the host binding rejects them)
  if (groups[3 * g] < 0 || groups[3 * g + 1] < 0 || groups[3 * g + 2] < 0 || gi >= gnx || gj >= gny || gk >= gnz) return;
  occ[((long long)gk * gny + gj) * gnx + gi] = g + 1;   // 0: not listed, else group index + 1
}

constexpr int kOccSmall = 16384;
__global__ void __launch_bounds__(1024) k_occ_small(int* occ, int cells, const int* groups, int n_groups,
                                                    const int* n_dev, int edge, int gnx, int gny, int gnz) {
  for (int t = threadIdx.x; t < cells; t += 1024) occ[t] = 0;
  const int n = n_dev ? min(*n_dev, n_groups) : n_groups;
  __syncthreads();
  for (int g = threadIdx.x; g < n; g += 1024) occ_set(occ, groups, g, edge, gnx, gny, gnz);
}

__global__ void __launch_bounds__(kBlock) k_occ_clear(int* occ, long long n) {
  const long long t = (long long)blockIdx.x * kBlock + threadIdx.x;
  if (t < n) occ[t] = 0;
}

__global__ void __launch_bounds__(kBlock) k_occ_set(int* occ, const int* groups, int n_groups, const int* n_dev,
                                                    int edge, int gnx, int gny, int gnz) {
  const int g = blockIdx.x * kBlock + threadIdx.x;
  const int n = n_dev ? min(*n_dev, n_groups) : n_groups;
  if (g < n) occ_set(occ, groups, g, edge, gnx, gny, gnz);
}

// ------------------------------------------------------------ set-up
template <typename T, bool MIX>
__global__ void __launch_bounds__(kBlock) k_prim_to_cons(Work w, const T* __restrict__ W5, const T* __restrict__ B,
                                                         T* __restrict__ U, Mix mix, T gam) {
  FOR_ITEMS(w, t) {
  int i, j, k;
  cell_of(w, t, i, j, k);
  const long long N = w.N;
  const long long p = lin(w, i, j, k);
  const T bx = T(0.5) * (B[p] + B[nbr(w, i, j, k, 1, 0, 0)]);
  const T by = T(0.5) * (B[N + p] + B[N + nbr(w, i, j, k, 0, 1, 0)]);
  const T bz = T(0.5) * (B[2 * N + p] + B[2 * N + nbr(w, i, j, k, 0, 0, 1)]);
  const T d = W5[p], vx = W5[N + p], vy = W5[2 * N + p], vz = W5[3 * N + p], pr = W5[4 * N + p];
  U[p] = d;
  U[N + p] = d * vx;
  U[2 * N + p] = d * vy;
  U[3 * N + p] = d * vz;
  if (MIX) {
    const double e = (double)pr / ((double)gam - 1.0) +
                     0.5 * (double)d * ((double)vx * vx + (double)vy * vy + (double)vz * vz) +
                     0.5 * ((double)bx * bx + (double)by * by + (double)bz * bz);
    mix.E64[p] = e;
    U[4 * N + p] = T(e);
  } else {
    U[4 * N + p] = pr / (gam - T(1)) + T(0.5) * d * (vx * vx + vy * vy + vz * vz) + T(0.5) * (bx * bx + by * by + bz * bz);
  }
  }
}

// ------------------------------------------------------------ diagnostics
// Two-pass deterministic reductions: a fixed number of blocks sum their cells
// through fixed trees, then one block per quantity combines the partials in index
// order and writes the result where the host reads it (pinned memory: no copy to
// wait for).  All three diagnostics on 128^3 in double, with their waits: 219 us with
// a block per 256 cells, one block for all rows of partials, 64-bit divisions for the
// cell and a copy of the result; 108 us so.
template <int NQ>
__device__ __forceinline__ void block_partials(double v[NQ], double* part, int stride) {
  __shared__ double red[NQ][kBlock / 64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const double s = wave_sum(v[q]);
    if (lane == 0) red[q][wid] = s;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      double s = red[q][0];
      for (int m = 1; m < kBlock / 64; ++m) s += red[q][m];
      part[(long long)q * stride + blockIdx.x] = s;
    }
  }
}

// discrete divergence (Eq. 16): partial sums of |div B| and partial maxima
template <typename T, int L>
__global__ void __launch_bounds__(kBlock) k_divb(Work w, const T* __restrict__ B, double inv_dx, double* part) {
  double a = 0.0, amax = 0.0;
  const long long N = w.N;
  FOR_CELLS(T, L, w, c) {
    const double bx = c.template level<0, 0>(w, B, 0), by = c.template level<0, 0>(w, B, N),
                 bz = c.template level<0, 0>(w, B, 2 * N);
    const double dv = ((double)c.template level<0, 1>(w, B, 0) - bx) * inv_dx +
                      ((double)c.template level<1, 1>(w, B, N) - by) * inv_dx +
                      ((double)c.template level<2, 1>(w, B, 2 * N) - bz) * inv_dx;
    a += fabs(dv);
    amax = fmax(amax, fabs(dv));
  }
  __shared__ double mx[kBlock / 64];
  const double wm = wave_max(amax);
  if ((threadIdx.x & 63) == 0) mx[threadIdx.x >> 6] = wm;
  double v[1] = {a};
  block_partials<1>(v, part, gridDim.x);
  if (threadIdx.x == 0) {
    double m = mx[0];
    for (int q = 1; q < kBlock / 64; ++q) m = fmax(m, mx[q]);
    part[(long long)gridDim.x + blockIdx.x] = m;
  }
}

// volume totals: mass, Mx, My, Mz, e, magnetic energy, kinetic energy
template <typename T, int L>
__global__ void __launch_bounds__(kBlock) k_sums(Work w, const T* __restrict__ U, const T* __restrict__ B,
                                                 const double* __restrict__ E64, double* part) {
  double v[7] = {0, 0, 0, 0, 0, 0, 0};
  const long long N = w.N;
  FOR_CELLS(T, L, w, c) {
    double u[5];
#pragma unroll
    for (int m = 0; m < 5; ++m) u[m] = (double)c.template level<0, 0>(w, U, m * N);
    const double bx = 0.5 * ((double)c.template level<0, 0>(w, B, 0) + (double)c.template level<0, 1>(w, B, 0));
    const double by = 0.5 * ((double)c.template level<0, 0>(w, B, N) + (double)c.template level<1, 1>(w, B, N));
    const double bz = 0.5 * ((double)c.template level<0, 0>(w, B, 2 * N) + (double)c.template level<2, 1>(w, B, 2 * N));
    if (E64) u[4] = E64[c.index(w)];
#pragma unroll
    for (int m = 0; m < 5; ++m) v[m] += u[m];
    v[5] += 0.5 * (bx * bx + by * by + bz * bz);
    v[6] += 0.5 * (u[1] * u[1] + u[2] * u[2] + u[3] * u[3]) / u[0];
  }
  block_partials<7>(v, part, gridDim.x);
}

// combine row blockIdx.x of nb partials (sum for rows < nsum, max otherwise)
__global__ void __launch_bounds__(kBlock) k_finish(const double* part, int nb, int nsum, double* out) {
  __shared__ double red[kBlock];
  const int q = blockIdx.x;
  const bool is_max = q >= nsum;
  double acc = 0.0;
  for (int b = threadIdx.x; b < nb; b += kBlock) {
    const double x = part[(long long)q * nb + b];
    acc = is_max ? fmax(acc, x) : acc + x;
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int s = kBlock / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] = is_max ? fmax(red[threadIdx.x], red[threadIdx.x + s])
                                                   : red[threadIdx.x] + red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[q] = red[0];
}

}  // namespace mhd
