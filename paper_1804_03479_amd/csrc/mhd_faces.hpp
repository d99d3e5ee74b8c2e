// mhd_faces.hpp -- the face kernels of CTU: step 1 (limited reconstruction and
// tracing) together with the Riemann fluxes of step 2, and again together with
// the transverse correction and the fluxes of steps 5-6.
//
// The kernels work line by line along each direction D.  A lane holds one line
// (y and z) and marches along it, keeping the stencil of five cells, the
// slopes and the interface value in registers: each cell is read once per
// direction, each slope and each interface value is computed once (a thread per
// cell computes them three and two times), the state above a face is there
// when the state below the next one is done, so the flux follows without a
// trip through memory, and the next cell's values are on their way while one
// is traced.  Along x the lanes are the line: a wave takes 64 successive cells
// of the rows and hands each upper-edge state to the next lane.
//
// The traced states are not kept: steps 5-6 trace again from the primitives
// (8 words a cell) instead of reading 42 words of stored states, which steps 1-2
// would have to write.
//
// With the learned flux (SOLVER 3) all 64 lanes of a wave meet at each face, so
// the network runs on the wave's 64 faces where a solver would run on each
// lane's.
//
// The work is cut into slabs -- rows and planes of a whole grid or of a listed
// group's item box -- and a slab into wave tasks: first the z-marches, then the
// y-marches, then the (short) x-rows, so that the short ones fill the end
// (face_geometry).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>

#include "mhd_kernels.hpp"

namespace mhd {

// Whether a march keeps what it carries from cell to cell -- slopes, interface
// values, the state below the next face: 21 words -- in LDS, each lane in slots of
// its own (no barrier), and reads the cells ahead again, instead of holding all of
// it in registers.  The Riemann solver then has the registers to itself: 72 / 96
// (steps 1-2 / 5-6, PPM + HLLD) instead of 142 / 160 in float, seven and five
// waves per SIMD instead of three; 139 / 162 and three waves instead of 256, spills
// and one wave in double.  128^3, steps 1-2 + 5-6: float 328 -> 292 us, double
// 1129 -> 788 us.  On group lists in float the cells read again miss the L2
// (many groups' boxes are in flight), so the registers keep them there: 337
// against 371 us for 191 groups (double 750 against 2200 us).
// The learned flux parks in both modes.
template <typename T, int SOLVER, bool L>
constexpr bool kPark = sizeof(T) == 8 || !L || SOLVER == 3;

// What a launch does with the traced states: take their fluxes (steps 1-2), or
// correct them first (steps 1, 5 and 6).
enum FaceStage { FACE_PREDICT = 1, FACE_CORRECT = 2 };

template <typename T>
struct FaceArgs {
  const T* W;      // primitives at time n
  const T* B;      // the level's face field at time n
  T* F;            // fluxes out
  const T* F1;     // FACE_CORRECT: predictor fluxes and EMFs, half-step face field
  const T* E1;
  const T* Bh;
  T gam;
  T dtdx, hr;             // dt/dx, half of it (set in the kernel)
  const MlpWeights* mw;   // learned flux: weights, fallback thresholds, capture
  float dp, drho;
  Capture cp;
};

// Small whole grids and most group lists (face_geometry) take z and y without marches
// too: a wave holds a tile of successive cells of neighbouring lines (columns along x), and hands each upper-edge
// state a row of lanes on.  A march of one cell traces two cells for each face, and too
// few waves are there to make it longer; a tile of eight traces eight for seven.  Fewer
// columns trace less and read shorter pieces of rows.  Whole step (us), 4 / 8 / 16
// columns: float HLLD 32^3 38 / 37 / 37, 64^3 103 / 78 / 73, 80^3 181 / 130 / 119, float
// Roe 64^3 106 / 98 / 100, double HLLD 48^3 85 / 82 / 89, 80^3 274 / 268 / 285, learned
// flux 64^3 156 / 159 / 167.
template <typename T, int SOLVER>
constexpr int kTileCols = sizeof(T) == 4 && (SOLVER == 1 || SOLVER == 2) ? 16 : 8;
template <typename T, int SOLVER>
constexpr int kTileCells = 64 / kTileCols<T, SOLVER>;

// value of the lane below (lane 0 keeps its own)
__device__ __forceinline__ float lane_below(float v) {
  const int x = __float_as_int(v);
  return __int_as_float(__builtin_amdgcn_update_dpp(x, x, 0x138, 0xf, 0xf, false));   // wave_shr:1
}
__device__ __forceinline__ double lane_below(double v) {
  const int lo = __double2loint(v), hi = __double2hiint(v);
  return __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, 0x138, 0xf, 0xf, false),
                          __builtin_amdgcn_update_dpp(lo, lo, 0x138, 0xf, 0xf, false));
}

__device__ __forceinline__ unsigned fresh_offset(unsigned o) {
  asm volatile("" : "+v"(o));
  return o;
}

// A lane's line along D (D = 1, 2), or its cell (D = 0): the byte offset of the
// line's position 0 (of the cell) in a component of the scratch, and the level
// index where the level is addressed apart from it (L).
template <typename T, int D, bool L>
struct Line {
  unsigned o;
  long long u;          // uniform element offset (L: the group's box)
  long long p;          // L: level index of the line without D's part
  int i, j, k;          // cell of the level (the coordinate along D left out)
  int g0;               // L: level coordinate of position 0 along D

  // element offset of position m along the line
  __device__ __forceinline__ long long step(const Work& w, int m) const {
    if constexpr (L) return u + (long long)m * (D == 1 ? w.sb : w.sb * w.sb);
    else if constexpr (D == 1) return (long long)wrapc(m, w.ny) * w.nx;
    else return (long long)wrapc(m, w.nz) * w.nx * w.ny;
  }
  // the level index of position m
  __device__ __forceinline__ long long index(const Work& w, int m) const {
    if constexpr (L)
      return p + (D == 1 ? (long long)wrapc(g0 + m, w.ny) * w.nx : (long long)wrapc(g0 + m, w.nz) * w.nx * w.ny);
    else return o / sizeof(T) + step(w, m);
  }
  // the level's B at position m
  __device__ __forceinline__ T face(const Work& w, const T* B, int m, unsigned off) const {
    if constexpr (L) {
      const long long q = D == 1 ? (long long)wrapc(g0 + m, w.ny) * w.nx : (long long)wrapc(g0 + m, w.nz) * w.nx * w.ny;
      return B[D * w.N + p + q];
    } else {
      return load_at<T>(scalar(B + (D * w.N + step(w, m))), off);
    }
  }
};

// A face is done: store its flux.  on: the lane has a face; every lane of a wave
// calls (the learned flux runs on the whole wave).  index: the face's cell in the
// level, for the learned flux's capture.
template <typename T, int D, int SOLVER>
__device__ __forceinline__ int emit_face(const Work& w, const FaceArgs<T>& A, MlpShared* sh, bool on, long long at,
                                         unsigned o0, const T wl[7], const T wr[7], T bn, long long index) {
  constexpr int n = D, t1 = (D + 1) % 3, t2 = (D + 2) % 3, d = 7 * D;
  const long long NS = w.NS;
  T f[7];
  int fb = 0;
  if constexpr (SOLVER == 3) {
    fb = mlp_or_hlld(*sh, on, wl, wr, bn, A.gam, A.dp, A.drho, f, A.cp, 3 * index + D);
    if (!on) return 0;
  } else {
    if (!on) return 0;
    fb = riemann<SOLVER>(wl, wr, bn, A.gam, f);
  }
  const unsigned o = fresh_offset(o0);
  store_at<T>(scalar(A.F + (d * NS + at)), o, f[0]);
  store_at<T>(scalar(A.F + ((d + 1 + n) * NS + at)), o, f[1]);
  store_at<T>(scalar(A.F + ((d + 1 + t1) * NS + at)), o, f[2]);
  store_at<T>(scalar(A.F + ((d + 1 + t2) * NS + at)), o, f[3]);
  store_at<T>(scalar(A.F + ((d + 4) * NS + at)), o, f[4]);
  store_at<T>(scalar(A.F + ((d + 5) * NS + at)), o, f[6]);    // E_t1 = F_n[B_t2]
  store_at<T>(scalar(A.F + ((d + 6) * NS + at)), o, -f[5]);   // E_t2 = -F_n[B_t1]
  return fb;
}

// o, o1, o2, o12: byte offsets of the cell and of its upper neighbours along t1,
// t2 and both (whole grid: wrapped; group boxes: d1 and d2 are the scalar
// distances instead and the offsets all equal)
template <typename T, int D>
__device__ __forceinline__ Transverse<T> transverse(const Work& w, const FaceArgs<T>& A, long long at, unsigned o,
                                                    unsigned o1, unsigned o2, unsigned o12, int d1, int d2) {
  constexpr int t1 = (D + 1) % 3, t2 = (D + 2) % 3;
  constexpr int comp[5] = {0, 1 + D, 1 + t1, 1 + t2, 4};
  const long long NS = w.NS;
  Transverse<T> r;
#pragma unroll
  for (int m = 0; m < 5; ++m) {
    const long long f1 = (7 * t1 + comp[m]) * NS + at, f2 = (7 * t2 + comp[m]) * NS + at;
    r.g[m] = A.hr * (load_at<T>(scalar(A.F1 + (f1 + d1)), o1) - load_at<T>(scalar(A.F1 + f1), o)) +
             A.hr * (load_at<T>(scalar(A.F1 + (f2 + d2)), o2) - load_at<T>(scalar(A.F1 + f2), o));
  }
  const long long ed = D * NS + at;
  const T e00 = load_at<T>(scalar(A.E1 + ed), o), e10 = load_at<T>(scalar(A.E1 + (ed + d1)), o1);
  const T e01 = load_at<T>(scalar(A.E1 + (ed + d2)), o2), e11 = load_at<T>(scalar(A.E1 + (ed + d1 + d2)), o12);
  r.c1 = A.hr * (T(0.5) * (e01 + e11) - T(0.5) * (e00 + e10));
  r.c2 = A.hr * (T(0.5) * (e10 + e11) - T(0.5) * (e00 + e01));
  return r;
}

// March along D from cell `start` to cell end - 1, emitting the lower faces of
// every cell but the first.  (o1, o2, o12): see transverse().  park: the lane's
// LDS slots (kPark), 64 apart: 0..6 s, 7..13 lo, 14..20 below.
template <typename T, int D, int RECON, bool ALLW, int SOLVER, int STAGE, bool L>
__device__ __forceinline__ int march_line(const Work& w, const FaceArgs<T>& A, const Line<T, D, L>& ln, unsigned o1,
                                          unsigned o2, unsigned o12, bool on, int start, int end, T* park,
                                          MlpShared* sh) {
  constexpr int t1 = (D + 1) % 3, t2 = (D + 2) % 3;
  constexpr int comp[7] = {0, 1 + D, 1 + t1, 1 + t2, 4, 5 + t1, 5 + t2};
  const long long NS = w.NS;
  const int d1 = L ? (t1 == 0 ? 1 : (t1 == 1 ? w.sb : w.sb * w.sb)) : 0;
  const int d2 = L ? (t2 == 0 ? 1 : (t2 == 1 ? w.sb : w.sb * w.sb)) : 0;
  const auto cell = [&](int m, unsigned o, T q[7]) {
    const long long at = ln.step(w, m);
#pragma unroll
    for (int c = 0; c < 7; ++c) q[c] = load_at<T>(scalar(A.W + (comp[c] * NS + at)), o);
  };
  const auto half_field = [&](int m, unsigned o) {
    return STAGE == FACE_CORRECT ? load_at<T>(scalar(A.Bh + (D * NS + ln.step(w, m))), o) : T(0);
  };
  int fb = 0;
  // q0 the traced cell, q1 the next, q2 the one after it; s the slope and lo the
  // lower interface value of q0 (PPM), or s its difference from the cell before
  // (PLM); below the state below q0's lower face
  constexpr bool parked = kPark<T, SOLVER, L>;
  T q0[7], q1[7], q2[7], s[7], lo[7], below[7];
  T bl, hl;
  {
    T z0[7], z1[7];
    const unsigned o = fresh_offset(ln.o);
    if (RECON == 1) cell(start - 2, o, z0);
    cell(start - 1, o, z1);
    cell(start, o, q0);
    cell(start + 1, o, q1);
    if (RECON == 1) cell(start + 2, o, q2);
    bl = ln.face(w, A.B, start, o);
    hl = half_field(start, o);
#pragma unroll
    for (int c = 0; c < 7; ++c) {
      if (RECON == 1) {
        s[c] = mc_slope2(z1[c], q0[c], q1[c]);
        lo[c] = ppm_interface(z1[c], q0[c], mc_slope2(z0[c], z1[c], q0[c]), s[c]);
      } else {
        s[c] = q0[c] - z1[c];
      }
      below[c] = T(0);
      if (parked) {
        park[64 * c] = s[c];
        park[64 * (7 + c)] = lo[c];
        park[64 * (14 + c)] = T(0);
      }
    }
  }
#pragma unroll 1
  for (int m = start; m < end; ++m) {
    T next[7], hi[7], sl[7], sr[7];
    const unsigned o = fresh_offset(ln.o);
    if constexpr (parked) {
      cell(m, o, q0);
      cell(m + 1, o, q1);
      if (RECON == 1) cell(m + 2, o, q2);
    } else {
      cell(m + (RECON == 1 ? 3 : 2), o, next);
    }
    const T bu = ln.face(w, A.B, m + 1, o);
    const T hu = half_field(m + 1, o);
#pragma unroll
    for (int c = 0; c < 7; ++c) {
      if (parked) {
        s[c] = park[64 * c];
        lo[c] = park[64 * (7 + c)];
      }
      if (RECON == 1) {
        const T s1 = mc_slope2(q0[c], q1[c], q2[c]);
        hi[c] = ppm_interface(q0[c], q1[c], s[c], s1);
        s[c] = s1;
        sl[c] = lo[c];
        sr[c] = hi[c];
        ppm_limit(q0[c], sl[c], sr[c]);
      } else {
        const T dp = q1[c] - q0[c];
        const T sc = minmod(s[c], dp);
        s[c] = dp;
        sl[c] = q0[c] - T(0.5) * sc;
        sr[c] = q0[c] + T(0.5) * sc;
      }
      if (parked) {
        park[64 * c] = s[c];
        if (RECON == 1) park[64 * (7 + c)] = hi[c];
      }
    }
    trace_edges<T, ALLW>(q0, bl, bu, A.dtdx, A.gam, sl, sr);
    if constexpr (STAGE == FACE_CORRECT) {
      const Transverse<T> tr = transverse<T, D>(w, A, ln.step(w, m), o, o1, o2, o12, d1, d2);
      const T hd = A.hr * (bu - bl);
      correct_state(tr, bl, hl, hd, A.gam, sl);
      correct_state(tr, bu, hu, hd, A.gam, sr);
    }
    if (parked) {
#pragma unroll
      for (int c = 0; c < 7; ++c) {
        below[c] = park[64 * (14 + c)];
        park[64 * (14 + c)] = sr[c];
      }
    }
    if (m > start)
      fb += emit_face<T, D, SOLVER>(w, A, sh, on, ln.step(w, m), ln.o, below, sl, STAGE == FACE_CORRECT ? hl : bl,
                                    SOLVER == 3 && A.cp.buf ? ln.index(w, m) : 0);
#pragma unroll
    for (int c = 0; c < 7; ++c) {
      if constexpr (!parked) {
        below[c] = sr[c];
        if (RECON == 1) lo[c] = hi[c];
        q0[c] = q1[c];
        if (RECON == 1) {
          q1[c] = q2[c];
          q2[c] = next[c];
        } else {
          q1[c] = next[c];
        }
      }
    }
    bl = bu;
    hl = hu;
  }
  return fb;
}

// Cells one per lane, their lower neighbours along D in the lane below (D = 0: 64
// successive cells of the x-rows) or a row of lanes below (tiles).  (o1, o2, o12): see
// transverse().
template <typename T, int D, int RECON, bool ALLW, int SOLVER, int STAGE, bool L>
__device__ __forceinline__ int row_faces(const Work& w, const FaceArgs<T>& A, const Line<T, D, L>& ln, unsigned o1,
                                         unsigned o2, unsigned o12, bool emit, MlpShared* sh) {
  constexpr int t1 = (D + 1) % 3, t2 = (D + 2) % 3;
  constexpr int comp[7] = {0, 1 + D, 1 + t1, 1 + t2, 4, 5 + t1, 5 + t2};
  const long long NS = w.NS;
  const int at = D == 0 ? ln.i : D == 1 ? ln.j : ln.k, size = D == 0 ? w.nx : D == 1 ? w.ny : w.nz;
  const unsigned stride = (D == 0 ? 1u : D == 1 ? (unsigned)w.nx : (unsigned)w.nx * (unsigned)w.ny) * (unsigned)sizeof(T);
  const auto off = [&](int x, unsigned o) {   // offset of the cell x along D
    if (L) return o;
    const int i = at + x;
    return o + (unsigned)(i < 0 ? x + size : (i >= size ? x - size : x)) * stride;
  };
  const auto slot = [&](int d) { return d == 0 ? 1 : d == 1 ? w.sb : w.sb * w.sb; };   // L: slots to the next cell
  const auto value = [&](const T* arr, long long e, int x, unsigned o) {
    return load_at<T>(scalar(arr + (e + ln.u + (L ? (long long)x * slot(D) : 0))), off(x, o));
  };
  T q[5][7], sl[7], sr[7];
  const unsigned o = fresh_offset(ln.o);
#pragma unroll
  for (int x = RECON == 1 ? -2 : -1; x <= (RECON == 1 ? 2 : 1); ++x)
#pragma unroll
    for (int c = 0; c < 7; ++c) q[x + 2][c] = value(A.W, comp[c] * NS, x, o);
  T bl, bu;
  if constexpr (L) {
    const T* face = A.B + D * w.N + ln.p;
    bl = face[0];
    bu = face[(long long)(at + 1 >= size ? 1 - size : 1) * (D == 0 ? 1 : D == 1 ? w.nx : (long long)w.nx * w.ny)];
  } else {
    bl = value(A.B, D * w.N, 0, o);
    bu = value(A.B, D * w.N, 1, o);
  }
  T hl = T(0), hu = T(0);
  if constexpr (STAGE == FACE_CORRECT) {
    hl = value(A.Bh, D * NS, 0, o);
    hu = value(A.Bh, D * NS, 1, o);
  }
  trace_cell<T, RECON, ALLW>(q, bl, bu, A.dtdx, A.gam, sl, sr);
  if constexpr (STAGE == FACE_CORRECT) {
    const Transverse<T> tr = transverse<T, D>(w, A, ln.u, o, o1, o2, o12, L ? slot(t1) : 0, L ? slot(t2) : 0);
    const T hd = A.hr * (bu - bl);
    correct_state(tr, bl, hl, hd, A.gam, sl);
    correct_state(tr, bu, hu, hd, A.gam, sr);
  }
#pragma unroll
  for (int c = 0; c < 7; ++c) sr[c] = D == 0 ? lane_below(sr[c]) : __shfl_up(sr[c], kTileCols<T, SOLVER>, 64);
  return emit_face<T, D, SOLVER>(w, A, sh, emit, ln.u, ln.o, sr, sl, STAGE == FACE_CORRECT ? hl : bl,
                                 L ? ln.p : (long long)(ln.o / sizeof(T)));
}

// The geometry read where it is used, from the kernel's argument segment (arguments lie
// in it as in a struct), of which k_ctu_faces keeps two dozen words: as an ordinary
// argument they are all loaded at its start and, over a hundred scalar registers, parked
// in vector lanes and fetched from there in the marches (16 of the 519 vector
// instructions a cell in float, steps 1-2; two so).
struct FaceKernelArgs {
  Work w;
  FaceGeo g;
};
typedef __attribute__((address_space(4))) const FaceGeo ConstGeo;
__device__ __forceinline__ const ConstGeo& face_geo() {
  auto* p = (__attribute__((address_space(4))) const char*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const ConstGeo*)(p + offsetof(FaceKernelArgs, g));
}
__device__ __forceinline__ unsigned fdiv(__attribute__((address_space(4))) const FastDiv& f, unsigned n) {
  return fdiv(FastDiv{f.m, f.s}, n);
}

// ALLW: trace waves moving away from an edge too (HLL-family solvers).  The
// double form is held to 168 registers (three waves per SIMD; it needs 173), with
// Roe, which would spill 90 words there, to 256.
// Bound by vector issue: 128^3 PPM + HLLD takes 112 / 180 us in float for steps
// 1-2 / 5-6 (a thread per cell and stored states: 257 / 185 us) and 266 / 522 us
// in double (545 / 385 us); PPM + Roe 183 / 239 and 441 / 823 us.  SOLVER 3, the
// learned flux (float only): 398 / 443 us against 417 / 536 us with states stored
// for kernels of their own, and 39 words a cell of scratch less.  (Stage events of
// mhd_profile_step.)
template <typename T, int RECON, bool ALLW, int SOLVER, int STAGE, bool L, bool TILES>
__global__ void __launch_bounds__(kBlock, sizeof(T) == 8 ? (SOLVER == 0 ? 2 : 3) : 1)
    k_ctu_faces(Work w, FaceGeo geo, FaceArgs<T> A, DtSrc dts, T inv_dx, unsigned long long* nfb) {
  A.dtdx = T(get_dt(dts)) * inv_dx;
  A.hr = T(0.5 * get_dt(dts)) * inv_dx;
  const unsigned lane = threadIdx.x & 63;
  unsigned units = (unsigned)geo.units;
  if constexpr (L) {
    if (w.n_dev) {
      const int m = *w.n_dev - w.gbase;
      const long long listed = (long long)m * geo.slabs;
      units = m < 0 ? 0u : listed < (long long)units ? (unsigned)listed : units;
    }
  }
  const unsigned waves = units * geo.per, in_block = blockDim.x >> 6;
  const unsigned blocks = (waves + in_block - 1) / in_block;
  // byte distance of the upper neighbour of coordinate i of n (stride in cells)
  const auto up = [](int i, int n, unsigned stride) {
    return (i + 1 >= n ? (unsigned)(1 - n) : 1u) * stride * (unsigned)sizeof(T);
  };
  const unsigned plane = (unsigned)w.nx * (unsigned)w.ny;
  __shared__ T parks[kPark<T, SOLVER, L> && !TILES ? kBlock * 21 : 1];
  MlpShared* sh = nullptr;
  if constexpr (SOLVER == 3) {
    __shared__ MlpShared shared;
    sh = &shared;
    mlp_load_weights(shared, A.mw);
  }
  T* park = parks + (threadIdx.x >> 6) * (64 * 21) + lane;
  int fb = 0;
  for (unsigned r = block_rank(); r < blocks; r += gridDim.x) {
    const ConstGeo& g = face_geo();
    const unsigned rank = w.rev ? blocks - 1 - r : r;
    const unsigned wave = __builtin_amdgcn_readfirstlane(rank * in_block + (threadIdx.x >> 6));
    if (wave >= waves) continue;
    const unsigned unit = fdiv(g.by_per, wave);
    unsigned t = wave - unit * g.per;
    const unsigned group = L ? fdiv(g.by_slabs, unit) : 0u, slab = unit - group * g.slabs;
    const unsigned row0 = L ? slab : fdiv(g.by_ux, slab), sz = fdiv(g.by_uy, row0);
    // the slab's first cell
    const int x0 = L ? 0 : (int)(slab - row0 * (unsigned)g.ux) * g.bx;
    const int y0 = (int)(row0 - sz * (unsigned)g.uy) * g.by, z0 = (int)sz * g.bz;
    const int bz = min((int)g.bz, (L ? w.box : w.nz) - z0), by = min((int)g.by, (L ? w.box : w.ny) - y0);
    int ox = 0, oy = 0, oz = 0;
    long long box = 0;
    if constexpr (L) {
      const int* og = w.groups + 3LL * (w.gbase + group);
      ox = og[0] - w.halo; oy = og[1] - w.halo; oz = og[2] - w.halo;
      box = (w.gbase + (int)group + 1LL) * w.sb * w.sb * w.sb;
    }
    const auto place = [&](auto& ln, int x, int y, int z, bool fx, bool fy, bool fz) {
      // (x, y, z): position in the unit; f*: the coordinate counts toward the offsets
      if constexpr (L) {
        ln.u = box;
        ln.i = wrapc(ox + x, w.nx); ln.j = wrapc(oy + y, w.ny); ln.k = wrapc(oz + z, w.nz);
        ln.o = (unsigned)(((z + w.soff) * w.sb + (y + w.soff)) * w.sb + (x + w.soff)) * (unsigned)sizeof(T);
        ln.p = (fx ? ln.i : 0) + (long long)(fy ? ln.j : 0) * w.nx + (long long)(fz ? ln.k : 0) * w.nx * w.ny;
      } else {
        ln.u = 0;
        ln.i = x; ln.j = y; ln.k = z;
        ln.p = 0;
        ln.o = (((unsigned)z * (unsigned)w.ny + (unsigned)y) * (unsigned)w.nx + (unsigned)x) * (unsigned)sizeof(T);
      }
    };
    if constexpr (TILES) {
      if (t < g.w2 + g.w1) {
        // position of the lines, one cell shared with the wave before: the lines of a
        // tile's columns, each (of a whole grid) with its last cell before the first;
        // columns are counted on from row to row
        constexpr unsigned cols = kTileCols<T, SOLVER>;
        const bool zdir = t < g.w2;
        const unsigned c0 = lane & (cols - 1), cell = lane / cols;
        const unsigned len = (unsigned)(zdir ? g.bz : g.by) + (L ? 0 : 1);   // a group box's lines start at their first cell
        const unsigned l = (zdir ? t : t - g.w2) * (kTileCells<T, SOLVER> - 1) + cell;
        const bool in = l < (zdir ? g.tz : g.ty) * len;
        const unsigned c = in ? l : 0, tile = zdir ? fdiv(g.by_lz, c) : fdiv(g.by_ly, c), q = c - tile * len;
        const unsigned col = tile * cols + c0;
        const bool on = in && col < (unsigned)g.bx * (unsigned)(zdir ? g.by : bz) && (L || !zdir || q <= (unsigned)bz);
        const unsigned at = on ? col : 0, other = fdiv(g.by_bx, at);
        const int x = (int)(at - other * (unsigned)g.bx);
        // the line's cell, wrapped where a line starts before the grid (lanes without one: the first)
        const int m = !on ? 0 : L ? (int)q : zdir ? wrapc(z0 + (int)q - 1, w.nz) : wrapc((int)q - 1, w.ny);
        const bool emit = on && cell > 0 && q > 0;
        if (zdir) {
          Line<T, 2, L> ln;
          place(ln, x, (int)other, m, true, true, true);
          const unsigned o1 = L ? ln.o : ln.o + up(ln.i, w.nx, 1), dy = L ? 0u : up(ln.j, w.ny, (unsigned)w.nx);
          fb += row_faces<T, 2, RECON, ALLW, SOLVER, STAGE, L>(w, A, ln, o1, ln.o + dy, o1 + dy, emit, sh);
        } else {
          Line<T, 1, L> ln;
          place(ln, x, m, z0 + (int)other, true, true, true);
          const unsigned o1 = L ? ln.o : ln.o + up(ln.k, w.nz, plane), dx = L ? 0u : up(ln.i, w.nx, 1);
          fb += row_faces<T, 1, RECON, ALLW, SOLVER, STAGE, L>(w, A, ln, o1, ln.o + dx, o1 + dx, emit, sh);
        }
        continue;
      }
    } else if (t < g.w2) {
      const unsigned chunk = fdiv(g.by_w2c, t), l = (t - chunk * g.w2c) * 64 + lane, n = (unsigned)(g.bx * by);
      const unsigned y = fdiv(g.by_bx, l), xs = l - y * (unsigned)g.bx;
      const bool on = l < n && (L || x0 + (int)xs < w.nx);
      const int x = x0 + (on ? (int)xs : 0), line = y0 + (on ? (int)y : 0);
      // marches start one cell early, at a group box's first cell there
      const int za = (int)chunk * g.cz, zb = za + g.cz < bz ? za + g.cz : bz;
      if (za >= bz || (t - chunk * g.w2c) * 64 >= n) continue;   // a remainder's
      Line<T, 2, L> ln;
      place(ln, x, line, 0, true, true, false);
      ln.g0 = oz;
      const unsigned o1 = L ? ln.o : ln.o + up(ln.i, w.nx, 1), dy = L ? 0u : up(ln.j, w.ny, (unsigned)w.nx);
      fb += march_line<T, 2, RECON, ALLW, SOLVER, STAGE, L>(w, A, ln, o1, ln.o + dy, o1 + dy, on,
                                                            z0 + za - (L && z0 + za == 0 ? 0 : 1), z0 + zb, park, sh);
      continue;
    }
    t -= g.w2;
    if (!TILES && t < g.w1) {
      const unsigned chunk = fdiv(g.by_w1c, t), l = (t - chunk * g.w1c) * 64 + lane, n = (unsigned)(g.bx * bz);
      const unsigned z = fdiv(g.by_bx, l), xs = l - z * (unsigned)g.bx;
      const bool on = l < n && (L || x0 + (int)xs < w.nx);
      const int x = x0 + (on ? (int)xs : 0), line = z0 + (on ? (int)z : 0);
      const int ya = (int)chunk * g.cy, yb = ya + g.cy < by ? ya + g.cy : by;
      if (ya >= by || (t - chunk * g.w1c) * 64 >= n) continue;
      Line<T, 1, L> ln;
      place(ln, x, 0, line, true, false, true);
      ln.g0 = oy;
      const unsigned o1 = L ? ln.o : ln.o + up(ln.k, w.nz, plane), dx = L ? 0u : up(ln.i, w.nx, 1);
      fb += march_line<T, 1, RECON, ALLW, SOLVER, STAGE, L>(w, A, ln, o1, ln.o + dx, o1 + dx, on,
                                                            y0 + ya - (L && y0 + ya == 0 ? 0 : 1), y0 + yb, park, sh);
      continue;
    }
    t -= g.w1;
    {
      // position of the rows, one lane shared with the wave before
      const unsigned l = t * 63 + lane, n = (unsigned)g.lx * (unsigned)g.by * (unsigned)bz;
      const unsigned c = l < n ? l : 0, row = fdiv(g.by_lx, c), q = c - row * (unsigned)g.lx;
      const unsigned z = fdiv(g.by_by, row), r = row - z * (unsigned)g.by;
      const bool on = l < n && r < (unsigned)by && (L || x0 + (int)q <= w.nx);
      const int y = y0 + (r < (unsigned)by ? (int)r : 0);
      const int x = L ? (int)q : wrapc(x0 + (int)q - 1, w.nx);
      Line<T, 0, L> ln;
      place(ln, x, y, z0 + (int)z, true, true, true);
      const unsigned o1 = L ? ln.o : ln.o + up(ln.j, w.ny, (unsigned)w.nx), dz = L ? 0u : up(ln.k, w.nz, plane);
      fb += row_faces<T, 0, RECON, ALLW, SOLVER, STAGE, L>(w, A, ln, o1, ln.o + dz, o1 + dz, on && lane > 0 && q > 0, sh);
    }
  }
  if (SOLVER == 0 || SOLVER == 3) block_count_atomic(fb, nfb);
}

// Interface capture of the shock-capturing solvers, apart from the face kernels
// (which it would cost registers): every sampled face's states, traced (and
// corrected) again, and the flux the face kernel has stored.
template <int D, int n, int RECON, bool ALLW, int L>
__device__ __forceinline__ void traced_states(const Work& w, const float* __restrict__ W, const float* __restrict__ B,
                                              const Cell<float, L>& c, float dtdx, float gam, float sl[7],
                                              float sr[7]) {
  float q[5][7];
  load_frame<float, D, n - 2, L>(w, W, c, q[0]);
  load_frame<float, D, n - 1, L>(w, W, c, q[1]);
  load_frame<float, D, n, L>(w, W, c, q[2]);
  load_frame<float, D, n + 1, L>(w, W, c, q[3]);
  load_frame<float, D, n + 2, L>(w, W, c, q[4]);
  trace_cell<float, RECON, ALLW>(q, c.template level<D, n>(w, B, D * w.N), c.template level<D, n + 1>(w, B, D * w.N),
                                 dtdx, gam, sl, sr);
}

template <int D, int RECON, bool ALLW, int STAGE, int L>
__device__ __forceinline__ void capture_sample(const Work& w, const FaceArgs<float>& A, const Cell<float, L>& c,
                                               const Capture& cp, long long face) {
  constexpr int t1 = (D + 1) % 3, t2 = (D + 2) % 3, d = 7 * D;
  float wl[7], wr[7], other[7];
  traced_states<D, -1, RECON, ALLW, L>(w, A.W, A.B, c, A.dtdx, A.gam, other, wl);
  traced_states<D, 0, RECON, ALLW, L>(w, A.W, A.B, c, A.dtdx, A.gam, wr, other);
  float bn;
  if constexpr (STAGE == FACE_CORRECT) {
    bn = c.here(w, A.Bh, D * w.NS);
    correct_states<float, D, L>(w, A.F1, A.E1, A.B, bn, c, A.hr, A.gam, wl, wr);
  } else {
    bn = c.template level<D, 0>(w, A.B, D * w.N);
  }
  const float f[7] = {c.here(w, A.F, d * w.NS),            c.here(w, A.F, (d + 1 + D) * w.NS),
                      c.here(w, A.F, (d + 1 + t1) * w.NS), c.here(w, A.F, (d + 1 + t2) * w.NS),
                      c.here(w, A.F, (d + 4) * w.NS),      -c.here(w, A.F, (d + 6) * w.NS),
                      c.here(w, A.F, (d + 5) * w.NS)};
  capture_face(cp, face, wl, wr, bn, f);
}

// A launch row (blockIdx.y) per direction, so that a wave's faces share their branch and
// one atomic takes all its records.  Whole grids: a thread per sampled face (L = kFlat;
// multiples of the stride that are D modulo 3 lie `stride` cells apart, or `stride` / 3
// with D = 0 alone).  Step with capture (us), cells of all faces looked at / so, CTU + PPM
// + HLLD: 128^3 stride 97 2027 / 614, stride 2 2837 / 1670; 16^3 stride 97 62 / 45.
// Group lists: a thread per cell of the item boxes, whose lowest
// faces are not the step's.
template <int D, int RECON, bool ALLW, int STAGE, int L>
__device__ __forceinline__ void capture_direction(const Work& w, const FaceArgs<float>& A, const Capture& cp) {
  if constexpr (L == kFlat) {
    const long long s = cp.stride, first = s % 3 == 0 || D == 0 ? 0 : (s % 3 == D ? s : 2 * s);
    if (s % 3 == 0 && D != 0) return;
    const long long step = s % 3 == 0 ? s / 3 : s;
    for (long long l = first / 3 + block_linear_id() * step; l < w.N; l += item_stride() * step)
      capture_sample<D, RECON, ALLW, STAGE, L>(w, A, Cell<float, L>(w, typename Cell<float, L>::AtCell{(unsigned)l}), cp,
                                               3 * l + D);
  } else {
    FOR_CELLS(float, L, w, c) {
      const long long face = 3 * c.index(w) + D;
      if (face % cp.stride == 0 && (D == 0 ? c.a : D == 1 ? c.b : c.c) != 0)
        capture_sample<D, RECON, ALLW, STAGE, L>(w, A, c, cp, face);
    }
  }
}

template <int RECON, bool ALLW, int STAGE, int L>
__global__ void __launch_bounds__(kBlock) k_capture(Work w, FaceArgs<float> A, DtSrc dts, float inv_dx, Capture cp) {
  A.dtdx = float(get_dt(dts)) * inv_dx;
  A.hr = float(0.5 * get_dt(dts)) * inv_dx;
  if (blockIdx.y == 0) capture_direction<0, RECON, ALLW, STAGE, L>(w, A, cp);
  else if (blockIdx.y == 1) capture_direction<1, RECON, ALLW, STAGE, L>(w, A, cp);
  else capture_direction<2, RECON, ALLW, STAGE, L>(w, A, cp);
}

}  // namespace mhd
